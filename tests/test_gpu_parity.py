"""GPU parity: the HIP path, called through the C ABI, against the CPU oracle on the same
seeded inputs.  Tile lists, masks, statistics and scores must match bit for bit; attention
outputs within the stated tolerances."""
import math
import sys

import numpy as np
import pytest
import torch

from oracle import oracle as vo
from paper_2605_30325_amd import veda
from paper_2605_30325_amd import workloads as wlm
from tests import harness as hz

pytestmark = pytest.mark.gpu


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def _full_check(wl, **kw):
    _say(f"[parity] {wl.name}: grid {wl.grid} heads {wl.heads} d {wl.head_dim} {wl.dtype}")
    run = hz.run_gpu_path(wl, **kw)
    assert torch.isfinite(run.out.float()).all(), "a real token was left unwritten or is not finite"
    for b in range(wl.batch):
        for h in range(wl.heads):
            st = hz.check_head(run, h, batch=b)
            _say(f"[parity] {wl.name} b{b} h{h} {tuple(run.shapes[h])}: {st}")
    return run


def test_tiny_config_everything():
    _full_check(wlm.WORKLOADS["tiny"])


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 64), ("f32", 128)])
def test_small_ragged_grids_all_shapes(dtype, d):
    # 6 heads cover the three tile shapes; every axis has a ragged tail for some shape
    wl = wlm.custom_workload(f"ragged_{dtype}_{d}", 6, d, dtype, (9, 10, 14), True, (25, 100), seed=11,
                             latent_dim=64 if d == 128 else 32)
    run = _full_check(wl)
    assert len({tuple(s) for s in run.shapes}) == 3


def test_batch_two_and_strided_input():
    wl = wlm.custom_workload("batch2", 3, 128, "bf16", (5, 8, 12), True, (30, 100), seed=12, batch=2)
    _full_check(wl)
    # [batch, N, heads, d] storage viewed as [batch, heads, N, d]: strides handed to the library
    dev = torch.device("cuda:0")
    shapes = wlm.tile_shapes(wl)
    q, _, _ = wlm.make_qkv(wl, dev)
    q_bnhd = q.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3)
    assert not q_bnhd.is_contiguous()
    plan = veda.Plan(wl.batch, wl.heads, wl.head_dim, wl.grid, shapes, wl.torch_dtype)
    a, _, _ = veda.veda_tile_layout(plan, q)
    b, _, _ = veda.veda_tile_layout(plan, q_bnhd)
    assert torch.equal(a.view(torch.int16), b.view(torch.int16))


@pytest.mark.parametrize("hidden,dp,relu,unit", [(0, 12, True, 0), (20, 12, True, 0), (131, 8, False, 0),
                                                  (260, 200, True, 0), (0, 12, True, 2), (131, 8, False, 2),
                                                  (260, 200, True, 2)])
def test_estimator_shapes_bit_exact(hidden, dp, relu, unit):
    # widths that are not multiples of the kernel's blocking, a single affine layer, no ReLU;
    # 135..180 tiles per head: several 64-row blocks and 128x128 score blocks, all with ragged tails.
    # unit = 2: the chains as scalar fmaf on the vector units (VEDA_OPT_FP32_CHAIN_UNIT), the form that
    # defines them; unit = 0: where the library's probe of this device put them (the matrix cores on gfx950)
    wl = wlm.custom_workload(f"mlp_{hidden}_{dp}", 2, 64, "f32", (10, 20, 36), True, (50, 100), seed=21,
                             latent_dim=dp)
    _say(f"[parity] {wl.name}: estimator 192 -> {hidden} -> {dp} relu={relu}")
    dev = torch.device("cuda:0")
    shapes = wlm.tile_shapes(wl)
    rng = np.random.default_rng(77 + hidden)
    first = hidden if hidden else dp

    def weights():
        w1 = rng.uniform(-0.1, 0.1, (wl.heads, 3 * wl.head_dim, first)).astype(np.float32)
        b1 = rng.uniform(-0.05, 0.05, (wl.heads, first)).astype(np.float32)
        if not hidden:
            return w1, b1, None, None
        return (w1, b1, rng.uniform(-0.2, 0.2, (wl.heads, hidden, dp)).astype(np.float32),
                rng.uniform(-0.05, 0.05, (wl.heads, dp)).astype(np.float32))

    wq, wk = weights(), weights()
    q, k, _ = wlm.make_qkv(wl, dev)
    plan = veda.Plan(wl.batch, wl.heads, wl.head_dim, wl.grid, shapes, wl.torch_dtype)
    if unit:
        plan.set_option(veda.VEDA_OPT_FP32_CHAIN_UNIT, unit)
        assert plan.chain_unit() == unit
    qt, vm, _ = veda.veda_tile_layout(plan, q, veda.VEDA_TOKEN_MAJOR)
    kt, _, _ = veda.veda_tile_layout(plan, k, veda.VEDA_TOKEN_MAJOR, want_mask=False)
    scale = hz.score_scale_of(wl)
    s, _ = veda.veda_tile_score(plan, qt, kt, vm, veda.Mlp(*wq, relu, dev), veda.Mlp(*wk, relu, dev), scale)
    torch.cuda.synchronize()
    for h in range(wl.heads):
        shape = tuple(int(x) for x in shapes[h])
        lat = []
        for x, w in ((q, wq), (k, wk)):
            z = vo.trippool(hz.to_f32_numpy(x[0, h]), wl.grid, shape)
            lat.append(vo.mlp(z, w[0][h], w[1][h], None if w[2] is None else w[2][h],
                              None if w[3] is None else w[3][h], relu))
        ref = vo.score(lat[0], lat[1], np.float32(scale))
        nt, soff = plan.tiles[h], plan.score_offset[h]
        got = s[0, soff:soff + nt * nt].view(nt, nt).cpu().numpy()
        assert np.array_equal(got.view(np.uint32), ref.view(np.uint32)), f"{wl.name} head {h}: scores not bit-exact"


def test_this_device_runs_the_fp32_chains_on_the_matrix_cores():
    """veda_plan_create probes the device: chains of v_mfma_f32_32x32x2_f32 against the fmaf chains they stand
    for (rounding, signed zeros, denormal sums and products).  On gfx950 every bit agrees, so plans use the
    matrix cores; were this to fail on another device or driver, the library would already have switched to
    the vector units by itself and every bit-exactness test would still hold."""
    wl = wlm.custom_workload("probe", 1, 64, "f32", (4, 8, 8), False, (1, 2), seed=5, latent_dim=4)
    plan = veda.Plan(wl.batch, wl.heads, wl.head_dim, wl.grid, wlm.tile_shapes(wl), wl.torch_dtype)
    assert plan.chain_unit() == veda.VEDA_CHAINS_MATRIX
    plan.set_option(veda.VEDA_OPT_FP32_CHAIN_UNIT, veda.VEDA_CHAINS_VECTOR)
    assert plan.chain_unit() == veda.VEDA_CHAINS_VECTOR
    plan.set_option(veda.VEDA_OPT_FP32_CHAIN_UNIT, 0)
    assert plan.chain_unit() == veda.VEDA_CHAINS_MATRIX
    with pytest.raises(RuntimeError):
        plan.set_option(veda.VEDA_OPT_FP32_CHAIN_UNIT, 3)


def test_projection_chains_of_odd_length_keep_signed_zeros():
    """Hidden width 5: the second layer's chains have an odd number of terms, so the last matrix-core
    instruction of each chain carries a padding term, which must leave a -0 accumulator as -0
    (bias -0, every product 1 * -0): the latents are -0 in the oracle and on the GPU."""
    wl = wlm.custom_workload("negzero", 1, 64, "f32", (4, 8, 8), False, (1, 2), seed=5, latent_dim=4)
    dev = torch.device("cuda:0")
    shapes = wlm.tile_shapes(wl)
    q, k, _ = wlm.make_qkv(wl, dev)
    plan = veda.Plan(wl.batch, wl.heads, wl.head_dim, wl.grid, shapes, wl.torch_dtype)
    qt, vm, _ = veda.veda_tile_layout(plan, q, veda.VEDA_TOKEN_MAJOR)
    kt, _, _ = veda.veda_tile_layout(plan, k, veda.VEDA_TOKEN_MAJOR, want_mask=False)
    w1 = np.zeros((1, 192, 5), np.float32)
    b1 = np.ones((1, 5), np.float32)
    w2 = np.full((1, 5, 4), -0.0, np.float32)
    b2 = np.full((1, 4), -0.0, np.float32)
    z = vo.trippool(hz.to_f32_numpy(q[0, 0]), wl.grid, (4, 4, 4))
    want = vo.mlp(z, w1[0], b1[0], w2[0], b2[0], True)
    assert np.all(want.view(np.uint32) == 0x80000000)
    phi = veda.Mlp(w1, b1, w2, b2, True, dev)
    _, ws = veda.veda_tile_score(plan, qt, kt, vm, phi, phi, 0.5)
    torch.cuda.synchronize()
    _, _, yq, yk = hz.score_intermediates(plan, phi, phi, ws)
    assert np.all(yq.cpu().numpy().view(np.uint32) == 0x80000000)
    assert np.all(yk.cpu().numpy().view(np.uint32) == 0x80000000)


@pytest.mark.parametrize("dtype,d,tile_tokens,grid,heads", [
    ("bf16", 128, 64, (5, 9, 13), 3), ("bf16", 64, 64, (3, 17, 30), 5), ("f32", 128, 64, (6, 7, 9), 3), ("f32", 64, 64, (1, 5, 67), 3),
    ("bf16", 128, 128, (5, 9, 13), 3), ("bf16", 64, 128, (17, 6, 7), 3),
    ("f32", 64, 64, (8, 40, 40), 20), ("bf16", 64, 128, (16, 96, 96), 6), ("bf16", 64, 128, (8, 80, 80), 6),   # enough workgroups for three launches
])
@pytest.mark.parametrize("want_tiles", [True, False])
def test_stage_one_in_one_launch_gives_the_same_bytes(dtype, d, tile_tokens, grid, heads, want_tiles):
    shapes = [(4, 4, 4), (1, 8, 8), (16, 2, 2)]
    shapes = np.asarray([shapes[h % 3] for h in range(heads)], np.int32) * np.asarray([tile_tokens // 64, 1, 1], np.int32)
    wl = wlm.custom_workload("one_launch", heads, d, dtype, grid, False, (50, 100), seed=47, batch=2)
    q, k, v = wlm.make_qkv(wl, torch.device("cuda:0"))
    k = k.transpose(1, 2).contiguous().transpose(1, 2)   # a stride of its own for each
    v = torch.cat([v, v], dim=3)[..., :d]
    plan = veda.Plan(2, heads, d, grid, shapes, wl.torch_dtype, tile_tokens=tile_tokens)
    r = veda.veda_tile_layout_path(plan, q, k, v, want_tiles=want_tiles)
    qt, vm, vc, zq = veda.veda_tile_layout_stats(plan, q, want_tiles=want_tiles)
    kt, _, _, zk = veda.veda_tile_layout_stats(plan, k, want_mask=False, want_tiles=want_tiles)
    vt, _, _ = veda.veda_tile_layout(plan, v, veda.VEDA_CHANNEL_MAJOR, want_mask=False)
    torch.cuda.synchronize()
    for name, want in (("qt", qt), ("kt", kt), ("vt", vt), ("vm", vm), ("vc", vc), ("zq", zq), ("zk", zk)):
        if want is None:
            assert r[name] is None
        else:
            assert torch.equal(r[name].view(torch.uint8), want.view(torch.uint8)), name


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("tiles", [1, 31, 32, 33, 63, 64, 65, 130])
def test_usual_estimator_sizes_bit_exact(d, tiles):
    """192 -> 64 -> 32 and 384 -> 128 -> 64, the sizes with a kernel of their own, around the rows a workgroup takes;
    with weights at other alignments, which the general kernel serves, the same latents."""
    wl = wlm.custom_workload("usual", 2, d, "f32", (4, 4, 4 * tiles), False, (1, 2), seed=tiles, latent_dim=d // 2, batch=2)
    dev = torch.device("cuda:0")
    q, k, _ = wlm.make_qkv(wl, dev)
    plan = veda.Plan(2, 2, d, wl.grid, wlm.tile_shapes(wl), wl.torch_dtype)
    _, vm, _, zq = veda.veda_tile_layout_stats(plan, q)
    _, _, _, zk = veda.veda_tile_layout_stats(plan, k, want_mask=False)
    rng = np.random.default_rng(tiles)
    w = [rng.uniform(-0.2, 0.2, s).astype(np.float32) for s in ((2, 3 * d, d), (2, d), (2, d, d // 2), (2, d // 2))]
    w[2][:, :, 0] = -0.0   # and a column of zeros
    w[3][:, 0] = -0.0
    for relu in (True, False):
        phi = veda.Mlp(*w, relu, dev)
        odd = veda.Mlp(*w, relu, dev)
        odd.w1 = torch.cat([torch.zeros(1, device=dev), phi.w1.reshape(-1)])[1:].view(phi.w1.shape)
        assert odd.w1.data_ptr() % 16 == 4
        s, ws = veda.veda_tile_score_stats(plan, zq, zk, phi, phi, 1.0)
        s2, _ = veda.veda_tile_score_stats(plan, zq, zk, odd, odd, 1.0)
        torch.cuda.synchronize()
        assert torch.equal(s.view(torch.int32), s2.view(torch.int32))
        for b in range(2):
            for h in range(2):
                args = (w[0][h], w[1][h], w[2][h], w[3][h], relu)
                lat = [vo.mlp(vo.trippool(hz.to_f32_numpy(x[b, h]), wl.grid, (4, 4, 4)), *args) for x in (q, k)]
                ref = vo.score(lat[0], lat[1], np.float32(1.0))
                off = plan.score_offset[h]
                got = s[b, off:off + tiles * tiles].view(tiles, tiles).cpu().numpy()
                assert np.array_equal(got.view(np.uint32), ref.view(np.uint32)), (relu, b, h)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("heads,tiles", [(64, 33), (65, 33), (97, 17)])
def test_usual_estimator_sizes_of_many_heads(d, heads, tiles):
    """768 workgroups of 16 rows, and more, from where a workgroup takes 32 or 64: the latents' scores are those of the general kernel,
    which serves weights at other alignments."""
    dev, batch = torch.device("cuda:0"), 2
    plan = veda.Plan(batch, heads, d, (4, 4, 4 * tiles), np.asarray([(4, 4, 4)] * heads, np.int32), torch.float32)
    gen = torch.Generator(device=dev).manual_seed(tiles)
    z = torch.randn(batch * plan.total_tiles, 3 * d, device=dev, generator=gen)
    phi, odd = (veda.Mlp(*[np.random.default_rng(heads).uniform(-0.2, 0.2, x).astype(np.float32)
                           for x in ((heads, 3 * d, d), (heads, d), (heads, d, d // 2), (heads, d // 2))], True, dev) for _ in range(2))
    odd.w1 = torch.cat([torch.zeros(1, device=dev), phi.w1.reshape(-1)])[1:].view(phi.w1.shape)
    got = [veda.veda_tile_score_stats(plan, z, z, e, e, 0.5)[0].view(torch.int32) for e in (phi, odd)]
    torch.cuda.synchronize()
    assert torch.equal(got[0], got[1])


@pytest.mark.parametrize("heads", [1, 63, 64, 65])
def test_scores_of_many_heads_on_either_unit(heads):
    """A score block finds its head among 64 at a time; heads of 160, 224 and 140 tiles, whose last blocks hold one or three
    times 32 columns, whole and not; the scores on the matrix cores are those on the vector units."""
    grid, dev = (5, 28, 64), torch.device("cuda:0")
    shapes = np.asarray([[[1, 8, 8], [4, 4, 4], [1, 1, 64]][h % 3] for h in range(heads)], np.int32)
    plan = veda.Plan(1, heads, 64, grid, shapes, torch.float32)
    gen = torch.Generator(device=dev).manual_seed(heads)
    z = torch.randn(plan.total_tiles, 192, device=dev, generator=gen)
    rng = np.random.default_rng(heads)
    phi = veda.Mlp(*[rng.uniform(-0.2, 0.2, x).astype(np.float32) for x in ((heads, 192, 64), (heads, 64), (heads, 64, 36), (heads, 36))],
                   True, dev)
    got = []
    for unit in (veda.VEDA_CHAINS_MATRIX, veda.VEDA_CHAINS_VECTOR):
        plan.set_option(veda.VEDA_OPT_FP32_CHAIN_UNIT, unit)
        got.append(veda.veda_tile_score_stats(plan, z, z, phi, phi, 0.5)[0].view(torch.int32))
    torch.cuda.synchronize()
    assert torch.equal(got[0], got[1])


def test_projection_and_score_chains_in_the_denormal_range():
    """Weights of magnitude 2^-136 (denormal themselves): every product and partial sum of the projection
    chains is a denormal number, and so are the latents; the scores underflow.  Nothing may be flushed to
    zero on the way: latents and scores have the oracle's bits (two layers and a single one)."""
    wl = wlm.custom_workload("denormal", 1, 64, "f32", (4, 8, 8), False, (1, 2), seed=6, latent_dim=8)
    dev = torch.device("cuda:0")
    shapes = wlm.tile_shapes(wl)
    q, k, _ = wlm.make_qkv(wl, dev)
    plan = veda.Plan(wl.batch, wl.heads, wl.head_dim, wl.grid, shapes, wl.torch_dtype)
    qt, vm, _ = veda.veda_tile_layout(plan, q, veda.VEDA_TOKEN_MAJOR)
    kt, _, _ = veda.veda_tile_layout(plan, k, veda.VEDA_TOKEN_MAJOR, want_mask=False)
    rng = np.random.default_rng(8)
    tiny = np.float32(2.0 ** -136)
    rows, d, dp = plan.total_tiles, 64, 8
    zq = vo.trippool(hz.to_f32_numpy(q[0, 0]), wl.grid, (4, 4, 4))
    zk = vo.trippool(hz.to_f32_numpy(k[0, 0]), wl.grid, (4, 4, 4))
    for hidden in (0, 12):
        first = hidden if hidden else dp
        w1 = (rng.uniform(-1, 1, (1, 3 * d, first)).astype(np.float32) * (tiny if not hidden else np.float32(1.0)))
        b1 = np.zeros((1, first), np.float32)
        w2 = rng.uniform(-1, 1, (1, hidden, dp)).astype(np.float32) * tiny if hidden else None
        b2 = rng.uniform(-1, 1, (1, dp)).astype(np.float32) * tiny if hidden else None
        args = (w1[0], b1[0], None if w2 is None else w2[0], None if b2 is None else b2[0], False)
        want_q, want_k = vo.mlp(zq, *args), vo.mlp(zk, *args)
        assert np.all(np.abs(want_q[want_q != 0]) < 1.1754944e-38) and np.count_nonzero(want_q) > want_q.size // 2
        phi = veda.Mlp(w1, b1, w2, b2, False, dev)
        s, ws = veda.veda_tile_score(plan, qt, kt, vm, phi, phi, 1.0)
        torch.cuda.synchronize()
        _, _, yq_g, yk_g = hz.score_intermediates(plan, phi, phi, ws)
        assert np.array_equal(yq_g.cpu().numpy().view(np.uint32), want_q.view(np.uint32)), hidden
        assert np.array_equal(yk_g.cpu().numpy().view(np.uint32), want_k.view(np.uint32)), hidden
        ref = vo.score(want_q, want_k, np.float32(1.0))
        assert np.array_equal(s[0].view(rows, rows).cpu().numpy().view(np.uint32), ref.view(np.uint32)), hidden
    # scores in the denormal range too: latents of magnitude 2^-68 give products near 2^-136
    w1 = rng.uniform(-1, 1, (1, 3 * d, dp)).astype(np.float32) * np.float32(2.0 ** -72)
    b1 = np.zeros((1, dp), np.float32)
    yq, yk = vo.mlp(zq, w1[0], b1[0], None, None, False), vo.mlp(zk, w1[0], b1[0], None, None, False)
    ref = vo.score(yq, yk, np.float32(1.0))
    assert np.count_nonzero(ref) > ref.size // 2 and np.all(np.abs(ref) < 1.1754944e-38)
    phi = veda.Mlp(w1, b1, None, None, False, dev)
    s, _ = veda.veda_tile_score(plan, qt, kt, vm, phi, phi, 1.0)
    torch.cuda.synchronize()
    assert np.array_equal(s[0].view(rows, rows).cpu().numpy().view(np.uint32), ref.view(np.uint32))


@pytest.mark.parametrize("n", [1, 2, 127, 128, 129, 257, 384, 385, 513, 641, 768, 769, 897, 1023, 1024, 1025, 1537, 2049, 3073, 4097])
def test_selection_of_every_row_length_class(n):
    """Row lengths around the registers a row takes; continuous scores (the search stops at the first cut), scores with many
    ties (it never finds one), one sign, and a few special values."""
    plan = veda.Plan(1, 1, 64, (4, 4, 4 * n), np.asarray([(4, 4, 4)], np.int32), torch.float32)
    g = torch.Generator(device="cuda").manual_seed(n)
    cont = torch.randn((n, n), device="cuda", generator=g)
    for scores in (cont, (cont * 4).round() / 4, cont.abs() + 1.0, torch.where(cont > 1.0, -0.0, torch.where(cont < -1.5, -math.inf, 0.0 * cont))):
        key = torch.where(scores == 0.0, 0.0, scores)
        order = torch.sort(key, dim=1, descending=True, stable=True)[1]
        for k in sorted({1, max(1, n // 20), max(1, n // 2), n}):
            _, ci = veda.veda_tile_select(plan, scores.reshape(1, -1).contiguous(), [k])
            assert torch.equal(ci.view(n, k).long(), torch.sort(order[:, :k], dim=1)[0]), (n, k)


def test_zero_sparsity_equals_dense_attention_on_gpu():
    wl = wlm.custom_workload("dense_identity", 3, 128, "bf16", (6, 9, 11), True, (1, 1), seed=13)
    run = hz.run_gpu_path(wl)
    assert list(run.k_per_head) == run.plan.tiles
    for h in range(wl.heads):
        qf, kf, vf = (hz.to_f32_numpy(t[0, h]) for t in (run.q, run.k, run.v))
        ref = vo.dense_attention(qf, kf, vf, run.softmax_scale, np.arange(wl.tokens))
        err = np.abs(hz.to_f32_numpy(run.out[0, h]).astype(np.float64) - ref)
        _say(f"[dense-identity] head {h} {tuple(run.shapes[h])}: max {err.max():.3e} mean {err.mean():.3e}")
        assert err.max() <= hz.BF16_MAX_ABS and err.mean() <= hz.BF16_MEAN_ABS


def test_row_stochastic_weights_on_gpu():
    # V == 1 everywhere: any convex combination of value rows is exactly 1 (bf16 can hold it)
    wl = wlm.custom_workload("ones", 3, 128, "bf16", (6, 9, 11), True, (40, 100), seed=14)
    run = hz.run_gpu_path(wl)
    vt, _, _ = veda.veda_tile_layout(run.plan, torch.ones_like(run.v), veda.VEDA_CHANNEL_MAJOR, want_mask=False)
    out, _ = veda.veda_sparse_attn_fwd(run.plan, run.bufs["qt"], run.bufs["kt"], vt, run.bufs["vm"],
                                       run.bufs["rp"], run.bufs["ci"], run.softmax_scale)
    torch.cuda.synchronize()
    assert (out.float() - 1.0).abs().max().item() <= 2 ** -7


@pytest.mark.parametrize("dtype,d,walk", [("bf16", 128, False), ("bf16", 64, False), ("f32", 64, False),
                                          ("bf16", 128, True), ("bf16", 64, True), ("f32", 64, True)])
def test_attention_on_hand_made_lists(dtype, d, walk):
    # Stage 4 alone on kept lists that stage 3 would never write: unsorted, neighbours with
    # identical / disjoint / partly shared lists.  The grid gives every head an odd tile count
    # (the last query tile has no neighbour) and ragged tiles on every axis.  walk: the kernel
    # merging the lists inside its loop (VEDA_OPT_ATTN_LIST_WALK) instead of from its step table.
    _hand_made_lists(dtype, d, 1.0, 1.0, walk=walk)


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 128), ("f32", 64)])
@pytest.mark.parametrize("grid,batch", [((9, 18, 18), 3), ((9, 18, 18), 6), ((9, 33, 33), 1), ((9, 33, 33), 2)])
def test_hand_made_lists_that_share_a_workgroup(dtype, d, grid, batch):
    """Calls whose tiles share workgroups: pairs, full and thin (711 and 757 tiles), and thin tiles in fours (1422 and 1514).  Unsorted lists of
    1 to 12 tiles, and all of them now and then, that are those of a neighbour along some axis in another order, share none
    of its tiles or a part: every tile against float64 softmax, from the step table and from lists merged in the loop."""
    dev, rng = torch.device("cuda:0"), np.random.default_rng(57)
    shapes = np.asarray([(4, 4, 4), (1, 8, 8), (16, 2, 2)], np.int32)
    wl = wlm.custom_workload("shared_lists", 3, d, dtype, grid, False, (25, 100), seed=59, batch=batch)
    q, k, v = wlm.make_qkv(wl, dev)
    plan = veda.Plan(batch, 3, d, grid, shapes, wl.torch_dtype)
    lists = []
    for h in range(3):
        nt, nh, nw = (-(-g // int(s)) for g, s in zip(grid, shapes[h]))
        n, of_head = nt * nh * nw, []
        for i in range(n):
            near = [i - step for step, at in ((nh * nw, i >= nh * nw), (nw, i // nw % nh), (1, i % nw)) if at]
            m, kind = int(rng.integers(1, 13)), int(rng.integers(0, 5))
            other = of_head[near[int(rng.integers(len(near)))]] if near else np.arange(0)
            if kind == 0 and len(other):
                own = rng.permutation(other)
            elif kind == 1 and len(other) < n:
                own = rng.choice(np.setdiff1d(np.arange(n), other), min(m, n - len(other)), replace=False)
            elif kind == 2 and len(other):
                own = rng.permutation(np.union1d(other[: (len(other) + 1) // 2], rng.choice(n, m, replace=False)))
            elif kind == 3 and i % 7 == 0:
                own = rng.permutation(n)
            else:
                own = rng.choice(n, m, replace=False)
            of_head.append(own)
        lists.append(of_head)
    flat = [x for of_head in lists for x in of_head]
    rp = torch.as_tensor(np.concatenate([[0], np.cumsum([len(x) for x in flat] * batch)]).astype(np.int32)).to(dev)
    ci = torch.as_tensor(np.concatenate(flat).astype(np.int32)).to(dev).repeat(batch)
    qt, vm, _ = veda.veda_tile_layout(plan, q)
    kt, _, _ = veda.veda_tile_layout(plan, k, want_mask=False)
    vt, _, _ = veda.veda_tile_layout(plan, v, veda.VEDA_CHANNEL_MAJOR, want_mask=False)
    scale, outs = 1.0 / math.sqrt(d), []
    for walk in (0, 1):
        plan.set_option(veda.VEDA_OPT_ATTN_LIST_WALK, walk)
        outs.append(veda.veda_sparse_attn_fwd(plan, qt, kt, vt, vm, rp, ci, scale, want_lse=True))
        torch.cuda.synchronize()
    peak, total, bar = 0.0, 0.0, (hz.BF16_MAX_ABS, 2e-2) if dtype == "bf16" else (hz.F32_MAX_ABS, 1e-4)
    for h in range(3):
        slots = _tile_tokens(tuple(int(x) for x in shapes[h]), grid)
        for i, kept in enumerate(lists[h]):
            rows, cols = slots[i][slots[i] >= 0].to(dev), slots[kept].reshape(-1)
            cols = cols[cols >= 0].to(dev)
            s = torch.matmul(q[:, h, rows].double(), k[:, h, cols].double().transpose(1, 2).contiguous()) * scale
            want, want_lse = torch.matmul(torch.softmax(s, dim=2), v[:, h, cols].double()), torch.logsumexp(s, dim=2)
            for out, lse in outs:
                err = (out[:, h, rows].double() - want).abs()
                worst = torch.stack([err.max() / bar[0], (lse[:, h, rows].double() - want_lse).abs().max() / bar[1], err.mean()]).tolist()
                assert max(worst[:2]) <= 1.0, (h, i, worst)
                peak, total = max(peak, worst[0]), total + worst[2]
    _say(f"[parity] shared lists {dtype} d {d} {grid} x {batch}: {peak:.2f} of the bar, mean {total / 2 / len(flat):.2e}")
    assert dtype == "f32" or total / 2 / len(flat) <= hz.BF16_MEAN_ABS


@pytest.mark.parametrize("exact_scale", [False, True])
@pytest.mark.parametrize("d,rows,cols", [(128, 16, 16), (128, 1, 257), (64, 16, 32), (64, 27, 19), (64, 1, 3)])
def test_lists_shared_by_the_wavefronts_of_a_tile(d, rows, cols, exact_scale):
    """Calls of few tiles, alone in their workgroups (up to 512) and in pairs; lists of one tile, of a few, odd ones, and all
    tiles (more steps than the table holds), one of them with an infinite key: against float64 softmax (bars of the bf16 path,
    logits of deviation 1), and the bits of the lists merged inside the loop."""
    dev, rng = torch.device("cuda:0"), np.random.default_rng(43)
    n, grid = rows * cols, (1, 8 * rows, 8 * cols - 3)   # the last column of tiles is ragged
    tokens = int(np.prod(grid))
    q, k, v = (torch.as_tensor(rng.standard_normal((1, 1, tokens, d), np.float32)).to(dev, torch.bfloat16) for _ in range(3))
    k[0, 0, -1, 3] = float("inf")   # of the last tile
    plan = veda.Plan(1, 1, d, grid, np.asarray([(1, 8, 8)], np.int32), torch.bfloat16)
    if exact_scale:
        plan.set_option(veda.VEDA_OPT_EXACT_LOGIT_SCALE, 1)
    vt, vm, _ = veda.veda_tile_layout(plan, v, veda.VEDA_CHANNEL_MAJOR)
    sizes = [min(s, n) for s in (1, 2, 7, 8, 9, 10, 33, n)]
    lists = [np.sort(rng.choice(n if i % 8 == 7 else max(1, n - 1), min(sizes[i % 8], n if i % 8 == 7 else n - 1), replace=False)) for i in range(n)]
    row_ptr = torch.as_tensor(np.concatenate([[0], np.cumsum([len(x) for x in lists])]).astype(np.int32)).to(dev)
    col_idx = torch.as_tensor(np.concatenate(lists).astype(np.int32)).to(dev)
    outs, scale = [], 1.0 / math.sqrt(d)
    for walk in (0, 1):
        plan.set_option(veda.VEDA_OPT_ATTN_LIST_WALK, walk)
        outs.append(veda.veda_sparse_attn_fwd(plan, None, None, vt, vm, row_ptr, col_idx, scale, want_lse=True, q_tokens=q, k_tokens=k))
        torch.cuda.synchronize()
    (out, lse), (out2, lse2) = outs
    assert torch.equal(out.view(torch.int16), out2.view(torch.int16)) and torch.equal(lse.view(torch.int32), lse2.view(torch.int32))
    h, w = torch.meshgrid(torch.arange(grid[1]), torch.arange(grid[2]), indexing="ij")
    tile_of = ((h // 8) * cols + w // 8).reshape(-1).to(dev)
    for i in list(range(min(n, 16))) + [n - 1]:
        rows_i, kept = (tile_of == i).nonzero()[:, 0], torch.isin(tile_of, torch.as_tensor(lists[i]).to(dev))
        s = (q[0, 0, rows_i].double() @ k[0, 0, kept].double().T) * scale
        want, want_lse = torch.softmax(s, dim=1) @ v[0, 0, kept].double(), torch.logsumexp(s, dim=1)
        err, fine = (out[0, 0, rows_i].double() - want).abs(), torch.isfinite(want_lse)
        assert bool((torch.isfinite(out[0, 0, rows_i].float()).all(dim=1) == fine).all()), i
        assert float(err[fine].max()) <= hz.BF16_MAX_ABS and float(err[fine].mean()) <= hz.BF16_MEAN_ABS, i
        assert float((lse[0, 0, rows_i].double() - want_lse)[fine].abs().max()) <= 2e-2, i


@pytest.mark.parametrize("dtype,d,exact_scale", [("bf16", 64, False), ("bf16", 128, False), ("bf16", 128, True), ("f32", 64, False), ("f32", 128, False)])
def test_a_sample_alone_and_in_a_batch(dtype, d, exact_scale):
    """176 tiles, thin ones among them, in calls of 1, 2, 3, 5, 6 and 40 samples (one tile to a workgroup, pairs, and thin tiles in
    fours): a sample's bits do not depend on how many others the call holds."""
    dev, heads, grid = torch.device("cuda:0"), 2, (5, 9, 61)
    wl = wlm.custom_workload("batch", heads, d, dtype, grid, False, (30, 100), seed=47)
    q, k, v = wlm.make_qkv(wl, dev)
    rng, shapes = np.random.default_rng(6), np.asarray([(4, 4, 4), (1, 8, 8)], np.int32)
    counts = veda.Plan(1, heads, d, grid, shapes, wl.torch_dtype).tiles
    lists = [np.sort(rng.choice(n, 20, replace=False)) for n in counts for _ in range(n)]
    first = None
    for batch in (1, 2, 3, 5, 6, 40):
        plan = veda.Plan(batch, heads, d, grid, shapes, wl.torch_dtype)
        if exact_scale:
            plan.set_option(veda.VEDA_OPT_EXACT_LOGIT_SCALE, 1)
        qb, kb, vb = (x.expand(batch, -1, -1, -1).contiguous() for x in (q, k, v))
        qt, vm, _ = veda.veda_tile_layout(plan, qb)
        kt, _, _ = veda.veda_tile_layout(plan, kb, want_mask=False)
        vt, _, _ = veda.veda_tile_layout(plan, vb, veda.VEDA_CHANNEL_MAJOR, want_mask=False)
        rp = torch.arange(batch * len(lists) + 1, dtype=torch.int32, device=dev) * 20
        ci = torch.as_tensor(np.concatenate(lists).astype(np.int32)).to(dev).repeat(batch)
        out, lse = veda.veda_sparse_attn_fwd(plan, qt, kt, vt, vm, rp, ci, 1.0 / math.sqrt(d), want_lse=True)
        torch.cuda.synchronize()
        first = first or (out[0].clone(), lse[0].clone())
        assert bool((out == first[0]).all()) and bool((lse == first[1]).all()), batch


@pytest.mark.parametrize("tile_tokens,rows,cols", [(64, 32, 64), (64, 3, 683), (128, 32, 64), (128, 3, 683)])
def test_step_table_up_to_and_past_a_word_a_lane(tile_tokens, rows, cols):
    """2048 tiles of a head, a bitmap word to each lane of a wavefront, and 2049, beyond it, with lists of one tile, of the
    last ones, and of more steps than the table holds at a time: the bits of the lists merged inside the loop."""
    grow = tile_tokens // 64
    grid, n, d = (grow, 8 * rows, 8 * cols - 3), rows * cols, 64   # the last column of tiles is ragged
    dev, rng = torch.device("cuda:0"), np.random.default_rng(41)
    q, k, v = (torch.as_tensor(rng.standard_normal((1, 1, int(np.prod(grid)), d), np.float32)).to(dev, torch.bfloat16) for _ in range(3))
    plan = veda.Plan(1, 1, d, grid, np.asarray([(grow, 8, 8)], np.int32), torch.bfloat16, tile_tokens=tile_tokens)
    vt, vm, _ = veda.veda_tile_layout(plan, v, veda.VEDA_CHANNEL_MAJOR)
    sizes = np.where(np.arange(n) % 97 == 0, 300, rng.integers(1, 6, n))
    lists = [np.sort(rng.choice(n, s, replace=False)) for s in sizes]
    lists[1], lists[2] = np.asarray([n - 1]), np.asarray([0, n - 2, n - 1])
    row_ptr = torch.as_tensor(np.concatenate([[0], np.cumsum([len(x) for x in lists])]).astype(np.int32)).to(dev)
    col_idx = torch.as_tensor(np.concatenate(lists).astype(np.int32)).to(dev)
    outs = []
    for walk in (0, 1):
        plan.set_option(veda.VEDA_OPT_ATTN_LIST_WALK, walk)
        outs.append(veda.veda_sparse_attn_fwd(plan, None, None, vt, vm, row_ptr, col_idx, 0.125, want_lse=True, q_tokens=q, k_tokens=k))
        torch.cuda.synchronize()
    assert bool(torch.isfinite(outs[0][0].float()).all())
    assert torch.equal(outs[0][0].view(torch.int16), outs[1][0].view(torch.int16)) and torch.equal(outs[0][1], outs[1][1])


def test_attention_with_large_logits_fp32():
    # Queries six times larger: logits spread over +-40 in log2 units, so the running softmax
    # reference moves on many steps and a stale one would overflow or flush rows to zero.
    _hand_made_lists("f32", 64, 6.0, 4.0)


def test_bf16_attention_error_against_logit_size():
    """Sweep of the query gain on the hand-made lists (logits q.k/sqrt(d) of standard deviation = gain).
    Default kernel: the pre-scaled queries are rounded to bf16 once, an error of 2^-9 of every logit, so the
    output error grows with the gain: the target's bars (max-abs 2e-2, mean-abs 2e-3) hold up to gain 2 and the
    measured growth stays inside the envelope the header documents.  With VEDA_OPT_EXACT_LOGIT_SCALE the
    bars hold at every gain, 6 (the large-logit case) and 16 included."""
    envelope = {1.0: (1e-2, 1e-3, 1e-2), 2.0: (2e-2, 2e-3, 2e-2), 4.0: (4e-2, 3e-3, 5e-2), 6.0: (8e-2, 4e-3, 1e-1),
                8.0: (1e-1, 4e-3, 1e-1)}
    for gain, (mx, mean, lse) in envelope.items():
        st = _hand_made_lists("bf16", 128, gain, 1.0, check=False)
        got = (max(s[0] for s in st), max(s[1] for s in st), max(s[2] for s in st))
        _say(f"[parity] default scale, gain {gain}: max_abs {got[0]:.2e} mean_abs {got[1]:.2e} lse {got[2]:.2e}")
        assert got[0] <= mx and got[1] <= mean and got[2] <= lse, (gain, got)
    for gain in (1.0, 2.0, 4.0, 6.0, 8.0, 16.0):
        st = _hand_made_lists("bf16", 128, gain, 1.0, check=True, exact_scale=True)
        got = (max(s[0] for s in st), max(s[1] for s in st), max(s[2] for s in st))
        _say(f"[parity] exact logit scale, gain {gain}: max_abs {got[0]:.2e} mean_abs {got[1]:.2e} lse {got[2]:.2e}")
    st = _hand_made_lists("bf16", 64, 6.0, 1.0, check=True, exact_scale=True)   # d = 64: residual factor 1.44


def _hand_made_lists(dtype, d, q_gain, tol_gain, check=True, exact_scale=False, walk=False):
    wl = wlm.custom_workload(f"lists_{dtype}_{d}", 3, d, dtype, (9, 18, 18), True, (25, 100), seed=31)
    dev = torch.device("cuda:0")
    shapes = wlm.tile_shapes(wl)
    q, k, v = wlm.make_qkv(wl, dev)
    q = (q.float() * q_gain).to(q.dtype)
    plan = veda.Plan(wl.batch, wl.heads, wl.head_dim, wl.grid, shapes, wl.torch_dtype)
    if exact_scale:
        plan.set_option(veda.VEDA_OPT_EXACT_LOGIT_SCALE, 1)
    if walk:
        plan.set_option(veda.VEDA_OPT_ATTN_LIST_WALK, 1)
    assert all(n % 2 for n in plan.tiles)
    qt, vm, _ = veda.veda_tile_layout(plan, q, veda.VEDA_TOKEN_MAJOR)
    kt, _, _ = veda.veda_tile_layout(plan, k, veda.VEDA_TOKEN_MAJOR, want_mask=False)
    vt, _, _ = veda.veda_tile_layout(plan, v, veda.VEDA_CHANNEL_MAJOR, want_mask=False)
    rng = np.random.default_rng(31)
    ksel = 7
    sels, cols = [], []
    for h in range(wl.heads):
        n = plan.tiles[h]
        sel = np.stack([rng.choice(n, ksel, replace=False) for _ in range(n)]).astype(np.int32)   # unsorted
        for i in range(0, n - 1, 2):
            kind = (i // 2) % 4
            if kind == 0:
                sel[i + 1] = sel[i][::-1]                                   # same tiles, other order
            elif kind == 1:
                rest = np.setdiff1d(np.arange(n), sel[i])
                sel[i + 1] = rng.choice(rest, ksel, replace=False)          # nothing shared
            elif kind == 2:
                sel[i], sel[i + 1] = np.sort(sel[i]), np.sort(sel[i + 1])   # ascending, as stage 3 writes
        sels.append(sel)
        cols.append(sel.reshape(-1))
    col_idx = torch.as_tensor(np.concatenate(cols)).to(dev)
    row_ptr = torch.arange(plan.total_tiles + 1, dtype=torch.int32, device=dev) * ksel
    scale = 1.0 / math.sqrt(d)
    out = torch.full((1, wl.heads, wl.tokens, d), float("nan"), dtype=wl.torch_dtype, device=dev)
    out, lse = veda.veda_sparse_attn_fwd(plan, qt, kt, vt, vm, row_ptr, col_idx, scale, out=out, want_lse=True)
    torch.cuda.synchronize()
    assert torch.isfinite(out.float()).all()
    queries = np.arange(wl.tokens)
    stats = []
    for h in range(wl.heads):
        shape = tuple(int(x) for x in shapes[h])
        ref, lse_ref, _ = vo.masked_attention(hz.to_f32_numpy(q[0, h]), hz.to_f32_numpy(k[0, h]),
                                              hz.to_f32_numpy(v[0, h]), wl.grid, shape, sels[h], scale, queries,
                                              want_stats=True)
        err = np.abs(hz.to_f32_numpy(out[0, h]).astype(np.float64) - ref)
        lerr = np.abs(lse[0, h].cpu().numpy().astype(np.float64) - lse_ref)
        _say(f"[parity] {wl.name} gain {q_gain} head {h} {shape}: max_abs {err.max():.2e} mean_abs {err.mean():.2e} "
             f"lse {lerr.max():.2e} (lse spread {lse_ref.max() - lse_ref.min():.1f})")
        stats.append((float(err.max()), float(err.mean()), float(lerr.max())))
        if not check:
            continue
        if dtype == "bf16":
            assert err.max() <= tol_gain * hz.BF16_MAX_ABS and err.mean() <= tol_gain * hz.BF16_MEAN_ABS
            assert lerr.max() <= tol_gain * 2e-2
        else:
            assert err.max() <= tol_gain * hz.F32_MAX_ABS and lerr.max() <= tol_gain * 1e-4
    return stats


def test_a_head_too_long_for_the_step_table():
    """1,049,600 tokens in one head = 17,600 tiles of 4x4x4, more than the 16,384 the bf16 attention kernel's
    step table covers: the kernel then merges the kept lists inside its loop.  Hand-made ascending lists (the
    tile itself, its successor, four drawn ones); sampled query tiles (first, last, ragged ones) against the
    oracle."""
    wl = wlm.custom_workload("long_head", 1, 64, "bf16", (41, 160, 160), False, (1, 100), seed=44)
    dev = torch.device("cuda:0")
    shapes = wlm.tile_shapes(wl)
    shape = tuple(int(x) for x in shapes[0])
    q, k, v = wlm.make_qkv(wl, dev)
    plan = veda.Plan(wl.batch, wl.heads, wl.head_dim, wl.grid, shapes, wl.torch_dtype)
    n = plan.tiles[0]
    assert n == 17600
    rng = np.random.default_rng(44)
    ksel = 6
    sel = np.empty((n, ksel), np.int32)
    sel[:, 0] = np.arange(n)
    sel[:, 1] = (np.arange(n) + 1) % n
    sel[:, 2:] = rng.integers(0, n, (n, ksel - 2))
    for i in range(n):   # no tile twice in a row: redraw the few duplicates
        while len(set(sel[i])) < ksel:
            sel[i, 2:] = rng.integers(0, n, ksel - 2)
    sel.sort(axis=1)
    col_idx = torch.as_tensor(sel.reshape(-1)).to(dev)
    row_ptr = torch.arange(n + 1, dtype=torch.int32, device=dev) * ksel
    _, vm, _, _ = veda.veda_tile_layout_stats(plan, q, want_tiles=False)
    vt, _, _ = veda.veda_tile_layout(plan, v, veda.VEDA_CHANNEL_MAJOR, want_mask=False)
    scale = 1.0 / math.sqrt(wl.head_dim)
    out = torch.full((1, 1, wl.tokens, wl.head_dim), float("nan"), dtype=wl.torch_dtype, device=dev)
    out, lse = veda.veda_sparse_attn_fwd(plan, None, None, vt, vm, row_ptr, col_idx, scale, out=out, want_lse=True,
                                         q_tokens=q, k_tokens=k)
    torch.cuda.synchronize()
    assert torch.isfinite(out.float()).all()
    T, H, W = wl.grid
    tiles = [0, 1, n // 2, n - 2, n - 1] + [int(x) for x in rng.integers(0, n, 3)]
    nh, nw = -(-H // shape[1]), -(-W // shape[2])
    queries = []
    for i in tiles:
        tt, th, tw = i // (nh * nw), (i // nw) % nh, i % nw
        for lt in range(shape[0]):
            for lh in range(shape[1]):
                for lw in range(shape[2]):
                    t, h, w = tt * shape[0] + lt, th * shape[1] + lh, tw * shape[2] + lw
                    if t < T and h < H and w < W:
                        queries.append((t * H + h) * W + w)
    queries = np.asarray(sorted(queries))
    ref, lse_ref, _ = vo.masked_attention(hz.to_f32_numpy(q[0, 0]), hz.to_f32_numpy(k[0, 0]), hz.to_f32_numpy(v[0, 0]),
                                          wl.grid, shape, sel, scale, queries, want_stats=True)
    got = hz.to_f32_numpy(out[0, 0][torch.as_tensor(queries, device=dev)]).astype(np.float64)
    err = np.abs(got - ref)
    lerr = np.abs(lse[0, 0][torch.as_tensor(queries, device=dev)].cpu().numpy().astype(np.float64) - lse_ref)
    _say(f"[parity] {wl.name}: {len(queries)} sampled queries of {n} tiles: max_abs {err.max():.2e} mean_abs {err.mean():.2e} "
         f"lse {lerr.max():.2e}")
    assert err.max() <= hz.BF16_MAX_ABS and err.mean() <= hz.BF16_MEAN_ABS and lerr.max() <= 2e-2


def test_maximum_head_count():
    # 128 heads (the library's limit) on a small ragged grid: per-head tables, the die-aware work
    # split and the 64-tile projection blocks all see many short heads
    wl = wlm.custom_workload("heads128", 128, 64, "bf16", (5, 6, 10), True, (50, 100), seed=41, latent_dim=16)
    run = hz.run_gpu_path(wl)
    assert torch.isfinite(run.out.float()).all()
    for h in (0, 1, 63, 126, 127):
        st = hz.check_head(run, h)
        _say(f"[parity] {wl.name} h{h} {tuple(run.shapes[h])}: {st}")
    with pytest.raises(veda.VedaError):
        veda.Plan(1, 129, 64, wl.grid, np.tile(np.asarray([[4, 4, 4]], np.int32), (129, 1)), torch.bfloat16)


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 64), ("f32", 128)])
def test_descriptors_during_gather_are_bit_identical(dtype, d):
    # veda_tile_layout_stats + veda_tile_score_stats against veda_tile_layout + veda_tile_score:
    # same tiled bytes, masks, descriptors (also checked against the oracle) and scores
    wl = wlm.custom_workload(f"fused_{dtype}_{d}", 5, d, dtype, (9, 10, 14), True, (25, 100), seed=51, batch=2,
                             latent_dim=32)
    dev = torch.device("cuda:0")
    shapes = wlm.tile_shapes(wl)
    q, k, _ = wlm.make_qkv(wl, dev)
    plan = veda.Plan(wl.batch, wl.heads, wl.head_dim, wl.grid, shapes, wl.torch_dtype)
    eq, ek = wlm.make_estimator(wl, "q"), wlm.make_estimator(wl, "k")
    pq = veda.Mlp(eq.w1, eq.b1, eq.w2, eq.b2, eq.relu, dev)
    pk = veda.Mlp(ek.w1, ek.b1, ek.w2, ek.b2, ek.relu, dev)
    scale = hz.score_scale_of(wl)
    qt, vm, vc = veda.veda_tile_layout(plan, q, veda.VEDA_TOKEN_MAJOR)
    kt, _, _ = veda.veda_tile_layout(plan, k, veda.VEDA_TOKEN_MAJOR, want_mask=False)
    s_ref, _ = veda.veda_tile_score(plan, qt, kt, vm, pq, pk, scale)
    qt2, vm2, vc2, zq = veda.veda_tile_layout_stats(plan, q)
    kt2, _, _, zk = veda.veda_tile_layout_stats(plan, k, want_mask=False)
    s2, _ = veda.veda_tile_score_stats(plan, zq, zk, pq, pk, scale)
    torch.cuda.synchronize()
    view = torch.int16 if dtype == "bf16" else torch.int32
    assert torch.equal(qt.view(view), qt2.view(view)) and torch.equal(kt.view(view), kt2.view(view))
    assert torch.equal(vm, vm2) and torch.equal(vc, vc2)
    assert torch.equal(s_ref.view(torch.int32), s2.view(torch.int32))
    for b in range(wl.batch):
        for h in range(wl.heads):
            shape = tuple(int(x) for x in shapes[h])
            nt, toff = plan.tiles[h], plan.tile_offset[h]
            for x, z in ((q, zq), (k, zk)):
                ref = vo.trippool(hz.to_f32_numpy(x[b, h]), wl.grid, shape)
                got = z[b, toff:toff + nt].cpu().numpy()
                assert np.array_equal(got.view(np.uint32), ref.view(np.uint32)), (b, h)


def test_select_on_constructed_ties_and_special_values():
    wl = wlm.custom_workload("ties", 2, 64, "f32", (4, 8, 40), False, (1, 4), seed=15, latent_dim=32)
    shapes = wlm.tile_shapes(wl)
    plan = veda.Plan(1, wl.heads, wl.head_dim, wl.grid, shapes, wl.torch_dtype)
    nt = plan.tiles[0]
    rng = np.random.default_rng(15)
    s = rng.integers(-2, 3, size=(wl.heads, nt, nt)).astype(np.float32)     # five levels: many ties
    s[0, 0, :5] = [np.nan, -0.0, 0.0, np.inf, -np.inf]
    s[1, 1, :] = 1.0                                                          # a fully tied row
    for k in (1, 3, nt // 2, nt):
        rp, ci = veda.veda_tile_select(plan, torch.as_tensor(s).reshape(1, -1).cuda(), [k] * wl.heads)
        torch.cuda.synchronize()
        got = ci.cpu().numpy().reshape(wl.heads, nt, k)
        for h in range(wl.heads):
            assert np.array_equal(got[h], vo.select(s[h], k)), (h, k)
        assert np.array_equal(rp.cpu().numpy(), np.arange(wl.heads * nt + 1) * k)


def test_select_long_rows_use_every_instantiation():
    # row lengths that land in the 4-, 16-, 32-, 64-item and the memory-resident kernels
    for grid in [(1, 8, 64), (32, 32, 64), (64, 32, 64), (128, 32, 64), (136, 32, 64)]:
        shapes = np.asarray([[1, 8, 8]], np.int32)
        plan = veda.Plan(1, 1, 64, grid, shapes, torch.float32)
        nt = plan.tiles[0]
        rows = min(nt, 48)
        s = np.random.default_rng(nt).standard_normal((nt, nt)).astype(np.float32)
        s[rows:] = 0.0
        # 5 % kept: rows of 1024 tiles and more take the sampled-pivot kernel; 50 % kept: the
        # register-resident (or memory-resident) full search
        for k in (max(1, nt // 20), nt // 2):
            _say(f"[parity] select grid {grid}: {nt} tiles, k {k}")
            rp, ci = veda.veda_tile_select(plan, torch.as_tensor(s).reshape(1, -1).cuda(), [k])
            torch.cuda.synchronize()
            got = ci.cpu().numpy().reshape(nt, k)
            assert np.array_equal(got[:rows], vo.select(s[:rows], k)), (grid, k)
            assert np.array_equal(got[rows:], np.tile(np.arange(k), (nt - rows, 1))), (grid, k)


@pytest.mark.parametrize("grid", [(1, 8, 64), (9, 18, 18), (136, 32, 64)])
def test_select_rows_of_one_sign_and_of_both(grid):
    """The search starts below the bits a row's scores share; the sign is the first of them.  Rows in registers and in
    memory, whole and ragged, with one sign, both, one value, two, and thresholds on either side of zero."""
    plan = veda.Plan(1, 1, 64, grid, np.asarray([[1, 8, 8]], np.int32), torch.float32)
    nt = plan.tiles[0]
    x = np.random.default_rng(nt).standard_normal((9, nt)).astype(np.float32)
    x[1], x[2] = np.abs(x[1]), -np.abs(x[2])
    x[3], x[4] = 3.0 + np.abs(x[3]) % 1.0, -3.0 - np.abs(x[4]) % 1.0       # many shared bits
    x[5], x[6] = -np.inf, np.where(x[6] > 0, np.inf, np.nan)
    x[7], x[8] = np.where(x[7] > 0, 2.0, -0.0), -1.0
    x[8, nt // 3] = 1.0                                                    # one of the other sign
    s = x[np.arange(nt) % 9]
    for k in sorted({1, nt // 2, nt - 1, nt} - {0}):
        _, ci = veda.veda_tile_select(plan, torch.as_tensor(s).reshape(1, -1).cuda(), [k])
        torch.cuda.synchronize()
        ref, got = vo.select(x, k), ci.cpu().numpy().reshape(nt, k)
        assert np.array_equal(got, ref[np.arange(nt) % 9]), (grid, k)


def test_select_sampled_pivot_paths():
    # 2048-tile rows at 5 % kept go through the sampled-pivot kernel.  Rows are built so that the
    # candidate list comes out well sized, too short (large values only where the sample looks),
    # too long (mass ties at the threshold), and with NaN / infinities / signed zeros in it.
    shapes = np.asarray([[1, 8, 8]], np.int32)
    plan = veda.Plan(1, 1, 64, (64, 32, 64), shapes, torch.float32)
    nt = plan.tiles[0]
    assert nt == 2048
    rng = np.random.default_rng(5)
    s = np.zeros((nt, nt), np.float32)
    rows = 40
    s[:8] = rng.standard_normal((8, nt))
    s[8:12] = rng.integers(-3, 4, size=(4, nt))                       # 7 levels: long tie runs
    s[12:16] = rng.standard_normal((4, nt))
    s[12:16, ::8] += 10.0                                             # the 256 sampled columns are the large ones
    s[16:20] = rng.standard_normal((4, nt))
    s[16:20, rng.integers(0, nt, 300)] = np.inf
    s[20:24] = rng.standard_normal((4, nt))
    s[20:24, rng.integers(0, nt, 1900)] = np.nan
    s[24:28] = np.where(rng.random((4, nt)) < 0.5, -0.0, 0.0)
    s[28:32] = -np.inf
    s[28:32, rng.integers(0, nt, 50)] = 1.0
    s[32:36] = rng.standard_normal((4, nt)).astype(np.float32) * 1e-30   # tiny values near the zero keys
    s[36:40] = -np.abs(rng.standard_normal((4, nt)))                  # all negative
    for k in (1, 64, 102, 180):
        _say(f"[parity] sampled select: k {k}")
        rp, ci = veda.veda_tile_select(plan, torch.as_tensor(s).reshape(1, -1).cuda(), [k])
        torch.cuda.synchronize()
        got = ci.cpu().numpy().reshape(nt, k)
        ref = vo.select(s[:rows], k)
        for r in range(rows):
            assert np.array_equal(got[r], ref[r]), (k, r)


def _lists_of(plan, stats_q, stats_k, pq, pk, sscale, kph):
    """(row_ptr, col_idx) by the two-stage route and by the one-call route, from descriptors."""
    s, _ = veda.veda_tile_score_stats(plan, stats_q, stats_k, pq, pk, sscale)
    rp, ci = veda.veda_tile_select(plan, s, kph)
    rp2, ci2, _ = veda.veda_tile_score_select(plan, pq, pk, sscale, kph, stats_q=stats_q, stats_k=stats_k)
    torch.cuda.synchronize()
    return (rp, ci), (rp2, ci2)


@pytest.mark.parametrize("hw", [(32, 32), (41, 25), (53, 29)])
def test_select_rows_whose_sample_is_one_value(hw):
    """Rows of 1024 tiles and more whose sampled columns are all alike skip the candidates: all equal, lower or higher
    in between, and the one value the lowest there is."""
    nt = hw[0] * hw[1]
    plan = veda.Plan(1, 1, 64, (1, 8 * hw[0], 8 * hw[1]), np.asarray([[1, 8, 8]], np.int32), torch.float32)
    sampled = np.arange(256) * nt // 256
    x = np.random.default_rng(nt).standard_normal((4, nt)).astype(np.float32)
    x[0] = 0.25
    x[1], x[2] = 0.25 - np.abs(x[1]), 0.25 + np.abs(x[2])
    x[:3, sampled] = 0.25
    x[3, sampled] = -np.inf
    s = torch.as_tensor(x[np.arange(nt) % 4]).reshape(1, -1).cuda()
    for k in (1, nt // 40, nt // 20):
        _say(f"[parity] select of {nt} tiles, one value sampled, k {k}")
        _, ci = veda.veda_tile_select(plan, s, [k])
        torch.cuda.synchronize()
        assert np.array_equal(ci.cpu().numpy().reshape(nt, k), vo.select(x, k)[np.arange(nt) % 4]), (nt, k)


def test_score_select_in_one_call_long_rows():
    # rows of 1260 - 1840 tiles at a 5 % budget: every score is compared with its row's pivot as it
    # is formed and never written.  Lists must equal the two-stage route's (which the other tests
    # hold against the oracle), from tiles and from descriptors; one head is checked against the
    # oracle directly as well.
    wl = wlm.custom_workload("one_call", 3, 128, "bf16", (21, 45, 80), True, (5, 100), seed=3)
    run = hz.run_gpu_path(wl)
    dev = torch.device("cuda:0")
    plan, kph = run.plan, run.k_per_head
    assert min(plan.tiles) >= 1024
    pq = veda.Mlp(run.phi_q.w1, run.phi_q.b1, run.phi_q.w2, run.phi_q.b2, run.phi_q.relu, dev)
    pk = veda.Mlp(run.phi_k.w1, run.phi_k.b1, run.phi_k.w2, run.phi_k.b2, run.phi_k.relu, dev)
    rp, ci, _ = veda.veda_tile_score_select(plan, pq, pk, run.score_scale, kph, q_tiled=run.bufs["qt"],
                                            k_tiled=run.bufs["kt"], valid_mask=run.bufs["vm"])
    torch.cuda.synchronize()
    assert torch.equal(rp, run.bufs["rp"]) and torch.equal(ci, run.bufs["ci"])
    _, _, _, zq = veda.veda_tile_layout_stats(plan, run.q)
    _, _, _, zk = veda.veda_tile_layout_stats(plan, run.k, want_mask=False)
    two, one = _lists_of(plan, zq, zk, pq, pk, run.score_scale, kph)
    assert torch.equal(two[0], run.bufs["rp"]) and torch.equal(two[1], run.bufs["ci"])
    assert torch.equal(one[0], run.bufs["rp"]) and torch.equal(one[1], run.bufs["ci"])
    st = hz.check_head(run, 0, attn_tiles=4)
    _say(f"[parity] {wl.name} head 0: lists equal on both routes and to the oracle; attention {st}")


@pytest.mark.parametrize("unit", [0, 2])
def test_score_select_in_one_call_ties_nan_and_redone_rows(unit):
    # Descriptors doctored against the candidate lists.  Head 0: every key tile is a copy of tile B
    # except 30 of the sampled columns, which are copies of tile A.  For a row that scores A above B
    # the pivot is A's score and only 30 < k candidates exist; for the other rows the pivot is B's
    # score and all 1152 > 1024 tiles pass: every row of the head is redone on its full score row,
    # all of it ties.  Head 1: key tiles are copies of six prototypes (whole runs of equal scores
    # around the k-th place, inside the candidate lists) and 40 of them hold NaN (rank as -inf).
    # Lists must equal the two-stage route's.
    wl = wlm.custom_workload("one_call_ties", 2, 64, "bf16", (16, 64, 72), False, (5, 100), seed=4, latent_dim=32)
    dev = torch.device("cuda:0")
    shapes = wlm.tile_shapes(wl)
    q, k, _ = wlm.make_qkv(wl, dev)
    plan = veda.Plan(wl.batch, wl.heads, wl.head_dim, wl.grid, shapes, wl.torch_dtype)
    if unit:   # projections and the redone score rows as scalar fmaf chains on the vector units
        plan.set_option(veda.VEDA_OPT_FP32_CHAIN_UNIT, unit)
    n = plan.tiles[0]
    assert n == 1152 and plan.tiles[1] == n
    kph = wlm.keep_budget(wl, None, shapes)
    assert int(kph[0]) == 58
    eq, ek = wlm.make_estimator(wl, "q"), wlm.make_estimator(wl, "k")
    pq = veda.Mlp(eq.w1, eq.b1, eq.w2, eq.b2, eq.relu, dev)
    pk = veda.Mlp(ek.w1, ek.b1, ek.w2, ek.b2, ek.relu, dev)
    _, _, _, zq = veda.veda_tile_layout_stats(plan, q)
    _, _, _, zk = veda.veda_tile_layout_stats(plan, k, want_mask=False)
    tile_a, tile_b = zk[0, 7].clone(), zk[0, 500].clone()
    zk[0, :n] = tile_b
    sampled = torch.as_tensor([(s * n) // 256 for s in range(30)], device=dev)
    zk[0, sampled] = tile_a
    g = torch.Generator(device="cpu").manual_seed(5)
    proto = torch.randint(0, 6, (n,), generator=g).to(dev)
    zk[0, n:2 * n] = zk[0, n:n + 6][proto]
    nan_at = torch.randperm(n, generator=g)[:40].to(dev) + n
    zk[0, nan_at, 0] = float("nan")
    sscale = hz.score_scale_of(wl)
    two, one = _lists_of(plan, zq, zk, pq, pk, sscale, kph)
    assert torch.equal(one[0], two[0]) and torch.equal(one[1], two[1])
    # the two-stage lists themselves against the oracle's selection on the same scores
    s, _ = veda.veda_tile_score_stats(plan, zq, zk, pq, pk, sscale)
    ksel = int(kph[0])
    for h in (0, 1):
        rows = s[0, h * n * n:(h + 1) * n * n].view(n, n)[[0, 1, n // 2, n - 1]].cpu().numpy()
        want = vo.select(rows, ksel)
        got = two[1][h * n * ksel:(h + 1) * n * ksel].view(n, ksel)[[0, 1, n // 2, n - 1]].cpu().numpy()
        assert np.array_equal(got, want), h
    a_first = (s[0, :n * n].view(n, n)[:, sampled[0]] > s[0, :n * n].view(n, n)[:, 1]).sum().item()
    _say(f"[parity] {wl.name}: head 0 redone in full ({a_first} rows short of candidates, {n - a_first} with too many)")


def test_score_select_in_one_call_other_shapes():
    # short rows, a large budget, 128-token tiles and a long latent: the call takes the two-stage
    # route inside and must give the same lists
    for tile_tokens, dp, keep in ((64, 64, (25, 100)), (128, 32, (25, 100)), (64, 128, (50, 100))):
        if tile_tokens == 64:
            wl = wlm.custom_workload("one_call_small", 3, 64, "bf16", (9, 18, 18), True, keep, seed=6, latent_dim=dp)
            shapes = wlm.tile_shapes(wl)
        else:
            shapes = np.asarray([(8, 4, 4), (2, 8, 8), (1, 8, 16)], np.int32)
            wl = wlm.custom_workload("one_call_128", 3, 64, "bf16", (9, 18, 18), True, keep, seed=6, latent_dim=dp)
        dev = torch.device("cuda:0")
        q, k, _ = wlm.make_qkv(wl, dev)
        plan = veda.Plan(wl.batch, wl.heads, wl.head_dim, wl.grid, shapes, wl.torch_dtype, tile_tokens=tile_tokens)
        kph = np.asarray([max(1, -(-n * keep[0] // keep[1])) for n in plan.tiles], np.int32)
        eq, ek = wlm.make_estimator(wl, "q"), wlm.make_estimator(wl, "k")
        pq = veda.Mlp(eq.w1, eq.b1, eq.w2, eq.b2, eq.relu, dev)
        pk = veda.Mlp(ek.w1, ek.b1, ek.w2, ek.b2, ek.relu, dev)
        qt, vm, _ = veda.veda_tile_layout(plan, q, veda.VEDA_TOKEN_MAJOR)
        kt, _, _ = veda.veda_tile_layout(plan, k, veda.VEDA_TOKEN_MAJOR, want_mask=False)
        sscale = hz.score_scale_of(wl)
        s, _ = veda.veda_tile_score(plan, qt, kt, vm, pq, pk, sscale)
        rp, ci = veda.veda_tile_select(plan, s, kph)
        rp2, ci2, ws = veda.veda_tile_score_select(plan, pq, pk, sscale, kph, q_tiled=qt, k_tiled=kt, valid_mask=vm)
        torch.cuda.synchronize()
        assert torch.equal(rp, rp2) and torch.equal(ci, ci2), (tile_tokens, dp)
        with pytest.raises(veda.VedaError) as e:
            veda.veda_tile_score_select(plan, pq, pk, sscale, kph, q_tiled=qt, k_tiled=kt, valid_mask=vm,
                                        workspace=ws[: ws.numel() // 2])
        assert e.value.status == veda.VEDA_ERR_WORKSPACE


@pytest.mark.parametrize("tile_tokens", [64, 128])
def test_whole_path_wrapper_routes_agree(tile_tokens):
    # veda_attention in its six routes (descriptors from the gather or not, stages 2+3 in one call
    # or two, Q and K tiled or read from token order): same lists, same output bits; buffers of a
    # first call are reused by a second.  With 128-token tiles the ragged grid leaves half tiles
    # without a single real token (8x4x4 on 9 frames, 1x8x16 on 18 columns).
    wl = wlm.custom_workload("routes", 3, 128, "bf16", (9, 18, 18), True, (25, 100), seed=12)
    dev = torch.device("cuda:0")
    shapes = wlm.tile_shapes(wl) if tile_tokens == 64 else np.asarray([(8, 4, 4), (2, 8, 8), (1, 8, 16)], np.int32)
    q, k, v = wlm.make_qkv(wl, dev)
    plan = veda.Plan(wl.batch, wl.heads, wl.head_dim, wl.grid, shapes, wl.torch_dtype, tile_tokens=tile_tokens)
    kph = wlm.keep_budget(wl, None, shapes)
    eq, ek = wlm.make_estimator(wl, "q"), wlm.make_estimator(wl, "k")
    pq = veda.Mlp(eq.w1, eq.b1, eq.w2, eq.b2, eq.relu, dev)
    pk = veda.Mlp(ek.w1, ek.b1, ek.w2, ek.b2, ek.relu, dev)
    outs = []
    for fused, one_call, from_tokens in ((False, False, False), (False, True, False), (True, False, False),
                                         (True, True, False), (True, False, True), (True, True, True)):
        out, bufs = veda.veda_attention(plan, q, k, v, pq, pk, kph, hz.score_scale_of(wl), 1.0 / math.sqrt(128),
                                        fused=fused, one_call=one_call, from_tokens=from_tokens)
        assert (bufs["qt"] is None and bufs["kt"] is None) == from_tokens
        first = out.clone()
        out2, _ = veda.veda_attention(plan, q, k, v, pq, pk, kph, hz.score_scale_of(wl), 1.0 / math.sqrt(128),
                                      buffers=bufs, fused=fused, one_call=one_call, from_tokens=from_tokens)
        torch.cuda.synchronize()
        assert out2.data_ptr() == out.data_ptr() and torch.equal(out2.view(torch.int16), first.view(torch.int16))
        outs.append((out2.view(torch.int16).clone(), bufs["ci"].clone(), bufs["vm"].clone(), bufs["vc"].clone(),
                     None if bufs.get("zq") is None or not fused else bufs["zq"].view(torch.int32).clone()))
    for o, ci, vm, vc, _ in outs[1:]:
        assert torch.equal(o, outs[0][0]) and torch.equal(ci, outs[0][1])
        assert torch.equal(vm, outs[0][2]) and torch.equal(vc, outs[0][3])     # masks and counts, from either gather
    # the descriptors of the gathers that write the tiles and of those that do not are the same bits
    assert torch.equal(outs[2][4], outs[4][4])
    # and they are the oracle's TripPool (Eq. 4) of every head
    zq = outs[2][4].view(torch.float32).cpu().numpy()
    for h in range(wl.heads):
        ref = vo.trippool(hz.to_f32_numpy(q[0, h]), wl.grid, tuple(int(x) for x in shapes[h]))
        got = zq[0, plan.tile_offset[h]:plan.tile_offset[h] + plan.tiles[h]]
        assert np.array_equal(got.view(np.uint32), ref.view(np.uint32)), (tile_tokens, h)


def test_whole_path_replayed_from_a_hip_graph():
    """The stage calls only enqueue kernels on the caller's stream, so one whole step can be captured into a
    HIP graph.  Replays with fresh inputs copied into the captured buffers, and unrelated eager work between
    them, must reproduce the eager results bit for bit every time."""
    wl = wlm.custom_workload("graph", 3, 128, "bf16", (9, 18, 18), True, (25, 100), seed=14)
    dev = torch.device("cuda:0")
    shapes = wlm.tile_shapes(wl)
    plan = veda.Plan(wl.batch, wl.heads, wl.head_dim, wl.grid, shapes, wl.torch_dtype)
    kph = wlm.keep_budget(wl, None, shapes)
    eq, ek = wlm.make_estimator(wl, "q"), wlm.make_estimator(wl, "k")
    pq = veda.Mlp(eq.w1, eq.b1, eq.w2, eq.b2, eq.relu, dev)
    pk = veda.Mlp(ek.w1, ek.b1, ek.w2, ek.b2, ek.relu, dev)
    args = (pq, pk, kph, hz.score_scale_of(wl), 1.0 / math.sqrt(128))
    kw = dict(fused=True, one_call=True, from_tokens=True)
    inputs = [wlm.make_qkv(wlm.custom_workload("graph", 3, 128, "bf16", (9, 18, 18), True, (25, 100), seed=14 + i), dev)
              for i in range(4)]
    q, k, v = (x.clone() for x in inputs[0])
    _, bufs = veda.veda_attention(plan, q, k, v, *args, **kw)        # allocates the step's buffers
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        veda.veda_attention(plan, q, k, v, *args, buffers=bufs, **kw)
    scratch = torch.zeros(1 << 20, device=dev)
    for rep, (qi, ki, vi) in enumerate(inputs[1:] + inputs[:1]):
        want, wb = veda.veda_attention(plan, qi, ki, vi, *args, **kw)   # eager, its own buffers
        want, want_ci = want.view(torch.int16).clone(), wb["ci"].clone()
        q.copy_(qi); k.copy_(ki); v.copy_(vi)
        scratch.add_(1.0).mul_(0.5)                                   # eager work between the replays
        bufs["out"].fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(bufs["ci"], want_ci), rep
        assert torch.equal(bufs["out"].view(torch.int16), want), rep


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_target_scores_replayed_from_a_hip_graph(dtype):
    """1920 work items on at most 1024 places: the counters they are drawn from are cleared by every replay, and the scratch, taken
    while the graph was recorded, stays the graph's own."""
    mk = lambda i: wlm.make_qkv(wlm.custom_workload("target_graph", 20, 128, dtype, (9, 32, 32), False, (25, 100), seed=17 + i), dev)[:2]
    dev, scale = torch.device("cuda:0"), 1.0 / math.sqrt(128)
    inputs = [mk(i) for i in range(3)]
    plan = veda.Plan(1, 20, 128, (9, 32, 32), np.asarray([(4, 4, 4)] * 20, np.int32), inputs[0][0].dtype)
    q, k = (x.clone() for x in inputs[0])
    qt, vm, vc = veda.veda_tile_layout(plan, q)
    kt, _, _ = veda.veda_tile_layout(plan, k, want_mask=False)
    heat = torch.zeros((1, plan.score_elems), device=dev)
    rp, ci = veda.veda_tile_select(plan, heat, [40] * 20)

    def step():
        veda.veda_tile_layout(plan, q, veda.VEDA_TOKEN_MAJOR, qt, vm, vc)
        veda.veda_tile_layout(plan, k, veda.VEDA_TOKEN_MAJOR, kt, want_mask=False)
        veda.veda_tile_heatmap(plan, qt, kt, vm, scale, None, heat)
        veda.veda_tile_select(plan, heat, [40] * 20, rp, ci)

    step()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    for rep, (qi, ki) in enumerate(inputs[1:] + inputs):
        q.copy_(qi); k.copy_(ki)
        step()
        want, want_ci = heat.clone(), ci.clone()
        other = torch.full((64 << 20,), 7.0, device=dev)   # would land in scratch that was given back
        heat.fill_(float("nan")); ci.zero_()
        graph.replay()
        other.add_(1.0)
        torch.cuda.synchronize()
        assert torch.equal(heat, want) and torch.equal(ci, want_ci), rep
        del other


@pytest.mark.parametrize("d,tile_tokens", [(128, 64), (64, 64), (128, 128)])
def test_attention_with_q_in_token_order(d, tile_tokens):
    # the attention kernel gathering Q itself (no tiled copy of Q): same bits as with the tiled Q; and
    # the descriptors-only gather gives the same descriptors and masks as the full one
    if tile_tokens == 64:
        wl = wlm.custom_workload(f"qtok_{d}", 3, d, "bf16", (9, 18, 18), True, (25, 100), seed=14, batch=2)
        shapes = wlm.tile_shapes(wl)
    else:
        shapes = np.asarray([(8, 4, 4), (2, 8, 8), (1, 8, 16)], np.int32)
        wl = wlm.custom_workload(f"qtok128_{d}", 3, d, "bf16", (9, 18, 18), True, (25, 100), seed=14, batch=2)
    dev = torch.device("cuda:0")
    q, k, v = wlm.make_qkv(wl, dev)
    plan = veda.Plan(wl.batch, wl.heads, d, wl.grid, shapes, wl.torch_dtype, tile_tokens=tile_tokens)
    qt, vm, _ = veda.veda_tile_layout(plan, q, veda.VEDA_TOKEN_MAJOR)
    kt, _, _ = veda.veda_tile_layout(plan, k, veda.VEDA_TOKEN_MAJOR, want_mask=False)
    vt, _, _ = veda.veda_tile_layout(plan, v, veda.VEDA_CHANNEL_MAJOR, want_mask=False)
    rng = np.random.default_rng(14)
    kph = [max(1, n // 4) for n in plan.tiles]
    cols = [np.sort(rng.choice(n, kk, replace=False)) for _ in range(wl.batch) for n, kk in zip(plan.tiles, kph)
            for _ in range(n)]
    col_idx = torch.as_tensor(np.concatenate(cols).astype(np.int32)).to(dev)
    lens = np.concatenate([[kk] * n for _ in range(wl.batch) for n, kk in zip(plan.tiles, kph)])
    row_ptr = torch.as_tensor(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)).to(dev)
    scale = 1.0 / math.sqrt(d)
    out1, lse1 = veda.veda_sparse_attn_fwd(plan, qt, kt, vt, vm, row_ptr, col_idx, scale, want_lse=True)
    # a strided view of Q: the gather must honour the strides
    qpad = torch.zeros((wl.batch, wl.heads, wl.tokens, d + 8), dtype=q.dtype, device=dev)
    qpad[..., :d] = q
    out2, lse2 = veda.veda_sparse_attn_fwd(plan, None, kt, vt, vm, row_ptr, col_idx, scale, want_lse=True,
                                           q_tokens=qpad[..., :d])
    # K from token order too, again through a strided view; the padded output starts as NaN so that a
    # real token left unwritten shows
    kpad = torch.zeros((wl.batch, wl.heads, wl.tokens, d + 8), dtype=k.dtype, device=dev)
    kpad[..., :d] = k
    out3 = torch.full_like(out1, float("nan"))
    out3, lse3 = veda.veda_sparse_attn_fwd(plan, None, None, vt, vm, row_ptr, col_idx, scale, out=out3, want_lse=True,
                                           q_tokens=qpad[..., :d], k_tokens=kpad[..., :d])
    torch.cuda.synchronize()
    assert torch.equal(out1.view(torch.int16), out2.view(torch.int16)) and torch.equal(lse1, lse2)
    assert torch.equal(out1.view(torch.int16), out3.view(torch.int16)) and torch.equal(lse1, lse3)
    # ascending rows: the lists merged inside the loop visit the key tiles in the step table's order
    plan.set_option(veda.VEDA_OPT_ATTN_LIST_WALK, 1)
    out4, lse4 = veda.veda_sparse_attn_fwd(plan, qt, kt, vt, vm, row_ptr, col_idx, scale, want_lse=True)
    out5 = torch.full_like(out1, float("nan"))
    out5, lse5 = veda.veda_sparse_attn_fwd(plan, None, None, vt, vm, row_ptr, col_idx, scale, out=out5, want_lse=True,
                                           q_tokens=qpad[..., :d], k_tokens=kpad[..., :d])
    plan.set_option(veda.VEDA_OPT_ATTN_LIST_WALK, 0)
    torch.cuda.synchronize()
    assert torch.equal(out1.view(torch.int16), out4.view(torch.int16)) and torch.equal(lse1, lse4)
    assert torch.equal(out1.view(torch.int16), out5.view(torch.int16)) and torch.equal(lse1, lse5)
    if tile_tokens == 64:
        _, vm_a, vc_a, z_a = veda.veda_tile_layout_stats(plan, q)
        none, vm_b, vc_b, z_b = veda.veda_tile_layout_stats(plan, q, want_tiles=False)
        torch.cuda.synchronize()
        assert none is None and torch.equal(vm_a, vm_b) and torch.equal(vc_a, vc_b)
        assert torch.equal(z_a.view(torch.int32), z_b.view(torch.int32)) and torch.equal(vm_a, vm)


def test_gpu_argument_errors_launch_nothing():
    wl = wlm.WORKLOADS["tiny"]
    run = hz.run_gpu_path(wl, want_lse=False)
    plan = run.plan
    with pytest.raises(veda.VedaError) as e:
        veda.veda_tile_select(plan, run.bufs["s"], [0, 2])
    assert e.value.status == veda.VEDA_ERR_INVALID_ARG
    with pytest.raises(veda.VedaError) as e:
        veda.veda_tile_select(plan, run.bufs["s"], [2, plan.tiles[1] + 1])
    assert e.value.status == veda.VEDA_ERR_INVALID_ARG
    pq = veda.Mlp(run.phi_q.w1, run.phi_q.b1, run.phi_q.w2, run.phi_q.b2)
    small = torch.empty(16, dtype=torch.uint8, device="cuda")
    with pytest.raises(veda.VedaError) as e:
        veda.veda_tile_score(plan, run.bufs["qt"], run.bufs["kt"], run.bufs["vm"], pq, pq, 0.125, workspace=small)
    assert e.value.status == veda.VEDA_ERR_WORKSPACE
    with pytest.raises(veda.VedaError) as e:
        veda.veda_sparse_attn_fwd(plan, run.bufs["qt"], run.bufs["kt"], run.bufs["vt"], run.bufs["vm"],
                                  run.bufs["rp"], run.bufs["ci"], float("nan"))
    assert e.value.status == veda.VEDA_ERR_INVALID_ARG


def test_outputs_are_deterministic():
    wl = wlm.custom_workload("determinism", 3, 128, "bf16", (6, 9, 11), True, (30, 100), seed=16)
    a, b = hz.run_gpu_path(wl), hz.run_gpu_path(wl)
    assert torch.equal(a.bufs["ci"], b.bufs["ci"]) and torch.equal(a.bufs["s"], b.bufs["s"])
    assert torch.equal(a.out.view(torch.int16), b.out.view(torch.int16))


def _default_route_matches(run):
    """The route bench.py times by default (descriptors from stats-only gathers of Q and K, stages 2+3 in
    one call, attention gathering Q and K rows from token order, only V tiled) against the stage-by-stage
    run that the oracle checks: same lists, same output bits."""
    wl, plan = run.wl, run.plan
    dev = run.q.device
    pq = veda.Mlp(run.phi_q.w1, run.phi_q.b1, run.phi_q.w2, run.phi_q.b2, run.phi_q.relu, dev)
    pk = veda.Mlp(run.phi_k.w1, run.phi_k.b1, run.phi_k.w2, run.phi_k.b2, run.phi_k.relu, dev)
    none_q, vm, _, zq = veda.veda_tile_layout_stats(plan, run.q, want_tiles=False)
    none_k, _, _, zk = veda.veda_tile_layout_stats(plan, run.k, want_mask=False, want_tiles=False)
    assert none_q is None and none_k is None and torch.equal(vm, run.bufs["vm"])
    rp, ci, _ = veda.veda_tile_score_select(plan, pq, pk, run.score_scale, run.k_per_head, stats_q=zq, stats_k=zk)
    out = torch.full_like(run.out, float("nan"))
    out, _ = veda.veda_sparse_attn_fwd(plan, None, None, run.bufs["vt"], vm, rp, ci, run.softmax_scale, out=out,
                                       q_tokens=run.q, k_tokens=run.k)
    torch.cuda.synchronize()
    assert torch.equal(rp, run.bufs["rp"]) and torch.equal(ci, run.bufs["ci"]), "kept lists differ"
    assert torch.equal(out.view(torch.int16), run.out.view(torch.int16)), "attention output differs"


def test_wan1p3b_480p_sampled():
    wl = wlm.WORKLOADS["wan1p3b_480p"]
    _say(f"[parity] {wl.name}")
    run = hz.run_gpu_path(wl)
    assert torch.isfinite(run.out.float()).all()
    for h in (0, 7):
        _say(f"[parity] {wl.name} head {h}: {hz.check_head(run, h, attn_tiles=12)}")
    _default_route_matches(run)


def _sampled_config(wl, keep=None, attn_tiles=6):
    """Full-size launch configuration; oracle on one head per tile shape and a seeded sample of
    query tiles (first and last tile always included)."""
    _say(f"[parity] {wl.name} keep {keep or wl.keep}: generating inputs")
    run = hz.run_gpu_path(wl, keep=keep, want_lse=False)
    for h in hz.heads_by_shape(run):
        _say(f"[parity] {wl.name} head {h} {tuple(run.shapes[h])} k {int(run.k_per_head[h])}: checking")
        _say(f"[parity] {wl.name} head {h}: {hz.check_head(run, h, attn_tiles=attn_tiles)}")
    # every real token of every head was written (the output buffer starts as NaN)
    for h in range(wl.heads):
        assert torch.isfinite(run.out[0, h].float()).all(), h
    _say(f"[parity] {wl.name}: the default route of bench.py against this run")
    _default_route_matches(run)


@pytest.mark.parametrize("name", ["wan14b_480p", "wan14b_720p", "waver12b_720p_241f"])
def test_large_configs_sampled(name):
    _sampled_config(wlm.WORKLOADS[name])


@pytest.mark.parametrize("keep", [(20, 100), (10, 100)])
def test_wan14b_720p_sparsity_sweep(keep):
    """The 80 % and 90 % points of the 75,600-token configuration's sparsity sweep (its 95 % point is the
    workload's default, above).  At these budgets stage 3 searches whole rows instead of sampling a pivot, and
    the one-call route of stages 2+3 goes through its two-stage path: both must still give the oracle's lists."""
    wl = wlm.WORKLOADS["wan14b_720p"]
    assert keep in wl.keep_sweep and wl.keep in wl.keep_sweep
    _sampled_config(wl, keep=keep, attn_tiles=4)


def test_waver12b_dense_heads_equal_full_attention():
    """0 % sparsity at 219,600 tokens: the full 24-head launch with k = N_T on the first head of every tile
    shape (the other heads keep their 5 %), against plain softmax attention over all tokens (Eq. 1) on sampled
    query tokens of the first and last tile and a seeded spread, and against the masked oracle on two tiles."""
    wl = wlm.WORKLOADS["waver12b_720p_241f"]
    shapes = wlm.tile_shapes(wl)
    kph = wlm.keep_budget(wl, None, shapes)
    nt = wlm.tiles_per_head(wl, shapes)
    dense_heads = []
    seen = set()
    for h, sh in enumerate(map(tuple, shapes)):
        if sh not in seen:
            seen.add(sh)
            dense_heads.append(h)
            kph[h] = nt[h]
    _say(f"[parity] {wl.name}: dense heads {dense_heads}, generating inputs")
    run = hz.run_gpu_path(wl, k_per_head=kph, want_lse=False)
    for h in range(wl.heads):
        assert torch.isfinite(run.out[0, h].float()).all(), h
    rng = np.random.default_rng(404)
    for h in dense_heads:
        shape = tuple(int(x) for x in shapes[h])
        tile_of = vo.token_tile_map(wl.grid, shape)
        first, last = np.flatnonzero(tile_of == 0), np.flatnonzero(tile_of == nt[h] - 1)
        queries = np.unique(np.concatenate([first[:24], last[-24:], rng.choice(wl.tokens, 80, replace=False)]))
        qf, kf, vf = (hz.to_f32_numpy(x[0, h]) for x in (run.q, run.k, run.v))
        ref = vo.dense_attention(qf, kf, vf, run.softmax_scale, queries)
        got = hz.to_f32_numpy(run.out[0, h])[queries].astype(np.float64)
        err = np.abs(got - ref)
        _say(f"[parity] {wl.name} dense head {h} {shape}: {len(queries)} tokens max_abs {err.max():.2e} "
             f"mean_abs {err.mean():.2e}")
        assert err.max() <= hz.BF16_MAX_ABS and err.mean() <= hz.BF16_MEAN_ABS
        # the kept lists are 0..N_T-1 on every row of a dense head
        r0 = run.plan.tile_offset[h]
        rp = run.bufs["rp"][r0:r0 + nt[h] + 1].cpu().numpy().astype(np.int64)
        assert np.all(np.diff(rp) == nt[h])
        for row in (0, int(nt[h]) // 2, int(nt[h]) - 1):
            lst = run.bufs["ci"][int(rp[row]):int(rp[row + 1])].cpu().numpy()
            assert np.array_equal(lst, np.arange(nt[h]))
    h = dense_heads[0]
    _say(f"[parity] {wl.name} dense head {h}: stages against the oracle, two tiles of masked attention")
    _say(f"[parity] {wl.name} dense head {h}: {hz.check_head(run, h, attn_tiles=2, check_layout=False)}")


@pytest.mark.parametrize("name", ["wan14b_720p", "waver12b_720p_241f"])
def test_128_token_tiles_at_full_size(name):
    """The paper's tile size at a named configuration's full launch size: every 64-token shape doubled along t
    (8x4x4, 2x8x8, 32x2x2), same kept fraction; one head per shape against the oracle on sampled tiles."""
    wl = wlm.WORKLOADS[name]
    shapes = wlm.tile_shapes(wl) * np.asarray([2, 1, 1], np.int32)
    kph = wlm.keep_budget(wl, None, shapes)
    _say(f"[parity] {wl.name} with 128-token tiles: generating inputs")
    run = hz.run_gpu_path(wl, k_per_head=kph, want_lse=False, shapes=shapes, tile_tokens=128)
    for h in hz.heads_by_shape(run):
        _say(f"[parity] {wl.name} head {h} {tuple(run.shapes[h])} k {int(kph[h])}: checking")
        _say(f"[parity] {wl.name} head {h}: {hz.check_head(run, h, attn_tiles=4)}")
    for h in range(wl.heads):
        assert torch.isfinite(run.out[0, h].float()).all(), h


@pytest.mark.parametrize("tile_tokens", [64, 128])
def test_list_walk_and_step_table_give_the_same_bits_at_full_size(tile_tokens):
    """wan14b_720p at its launch size: stage 3 writes ascending rows, so the attention kernel visits the key
    tiles in the same order whether it lays its steps out in LDS first or merges the lists inside its loop
    (VEDA_OPT_ATTN_LIST_WALK): every output bit agrees, from tiled K and Q and from token order."""
    wl = wlm.WORKLOADS["wan14b_720p"]
    shapes = wlm.tile_shapes(wl) * (np.asarray([2, 1, 1], np.int32) if tile_tokens == 128 else 1)
    run = hz.run_gpu_path(wl, k_per_head=wlm.keep_budget(wl, None, shapes), shapes=shapes, tile_tokens=tile_tokens)
    b, plan = run.bufs, run.plan
    args = (b["vt"], b["vm"], b["rp"], b["ci"], run.softmax_scale)
    outs = []
    for walk in (0, 1):
        plan.set_option(veda.VEDA_OPT_ATTN_LIST_WALK, walk)
        o1, l1 = veda.veda_sparse_attn_fwd(plan, b["qt"], b["kt"], *args, want_lse=True)
        o2, l2 = veda.veda_sparse_attn_fwd(plan, None, None, *args, want_lse=True, q_tokens=run.q, k_tokens=run.k)
        torch.cuda.synchronize()
        outs.append((o1, l1, o2, l2))
    plan.set_option(veda.VEDA_OPT_ATTN_LIST_WALK, 0)
    for x, y in zip(outs[0], outs[1]):
        assert torch.equal(x.view(torch.int16) if x.dtype == torch.bfloat16 else x, y.view(torch.int16) if y.dtype == torch.bfloat16 else y)
    assert torch.equal(outs[0][0].view(torch.int16), run.out.view(torch.int16))
    assert torch.equal(outs[0][0].view(torch.int16), outs[0][2].view(torch.int16))


@pytest.mark.parametrize("dtype,d,tile_tokens", [("bf16", 128, 64), ("bf16", 64, 64), ("bf16", 128, 128), ("bf16", 64, 128),
                                                  ("f32", 128, 64), ("f32", 64, 64)])
@pytest.mark.parametrize("grid", [(5, 9, 13), (17, 6, 7), (2, 3, 66), (1, 1, 1), (4, 57, 32)])
def test_edge_tiles_of_every_fill(dtype, d, tile_tokens, grid):
    """Key tiles with one to eight of their eight 8-slot chunks in use (half steps gather up to four of them,
    halves of 128-token tiles may hold nothing) and query tiles with fewer real rows than waves: outputs
    against the oracle, and the same bits from token order and from the walk inside the loop.  The last grid
    makes more steps than the table holds at a time (128)."""
    shapes = [(4, 4, 4), (1, 8, 8), (16, 2, 2), (2, 4, 8), (64, 1, 1), (1, 1, 64), (8, 8, 1)]
    if tile_tokens == 128:
        shapes = [(2 * a, b, c) for a, b, c in shapes]
    wl = wlm.custom_workload(f"edges_{d}", len(shapes), d, dtype, grid, False, (60, 100), seed=23, latent_dim=64 if d == 128 else 32)
    run = hz.run_gpu_path(wl, k_per_head=wlm.keep_budget(wl, None, np.asarray(shapes)), shapes=shapes, tile_tokens=tile_tokens)
    for h in range(wl.heads):
        hz.check_head(run, h, check_layout=False)
    if dtype == "bf16":
        _default_route_matches(run)
    b = run.bufs
    run.plan.set_option(veda.VEDA_OPT_ATTN_LIST_WALK, 1)
    for q, k in ((None, None), (run.q, run.k))[:2 if dtype == "bf16" else 1]:
        out, lse = veda.veda_sparse_attn_fwd(run.plan, b["qt"] if q is None else None, b["kt"] if k is None else None, b["vt"], b["vm"],
                                             b["rp"], b["ci"], run.softmax_scale, want_lse=True, q_tokens=q, k_tokens=k)
        torch.cuda.synchronize()
        assert np.array_equal(hz.raw_numpy(out), hz.raw_numpy(run.out)) and torch.equal(lse, run.lse)


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 128)])
@pytest.mark.parametrize("grid,batch", [((5, 9, 26), 1), ((5, 9, 13), 2)])
def test_thin_tiles_in_pairs(dtype, d, grid, batch):
    """Calls of 514 and 570 tiles in 260 and 290 workgroups, most of them pairs of thin tiles: two wavefronts, of a die's workgroups past the
    32nd (first grid) the other two.  Outputs against the oracle, and the bits of the walk inside the loop."""
    shapes = [(4, 4, 4), (1, 8, 8), (16, 2, 2), (2, 4, 8), (64, 1, 1), (1, 1, 64), (8, 8, 1)]
    heads = len(shapes)
    wl = wlm.custom_workload(f"thin_pairs_{d}", heads, d, dtype, grid, False, (60, 100), seed=29, batch=batch, latent_dim=64 if d == 128 else 32)
    run = hz.run_gpu_path(wl, k_per_head=wlm.keep_budget(wl, None, np.asarray(shapes)), shapes=shapes)
    for h in range(heads):
        hz.check_head(run, h, check_layout=False)
    b = run.bufs
    run.plan.set_option(veda.VEDA_OPT_ATTN_LIST_WALK, 1)
    out, lse = veda.veda_sparse_attn_fwd(run.plan, b["qt"], b["kt"], b["vt"], b["vm"], b["rp"], b["ci"], run.softmax_scale, want_lse=True)
    torch.cuda.synchronize()
    assert np.array_equal(hz.raw_numpy(out), hz.raw_numpy(run.out)) and torch.equal(lse, run.lse)


def test_rows_three_times_longer_than_any_named_workload():
    """783,360 tokens in one head (12,240 tiles per score row): the whole path against the oracle at a 2 %
    budget (stages 2+3 in one call take the candidate route), then the lists at a 5 % budget (k = 612, where
    that call falls back to the two stages) against the oracle's selection on the same, already checked, scores."""
    wl = wlm.custom_workload("long_video", 1, 128, "bf16", (96, 68, 120), False, (2, 100), seed=31)
    _say(f"[parity] {wl.name}: generating inputs")
    run = hz.run_gpu_path(wl, want_lse=False)
    assert run.plan.tiles[0] == 12240 and int(run.k_per_head[0]) == 245
    _say(f"[parity] {wl.name}: checking against the oracle")
    _say(f"[parity] {wl.name}: {hz.check_head(run, 0, attn_tiles=4)}")
    assert torch.isfinite(run.out.float()).all()
    _default_route_matches(run)

    _say(f"[parity] {wl.name}: 5 % budget")
    k5 = wlm.keep_budget(wl, (5, 100), run.shapes)
    assert int(k5[0]) == 612
    rp2, ci2 = veda.veda_tile_select(run.plan, run.bufs["s"], k5)
    dev = run.q.device
    pq = veda.Mlp(run.phi_q.w1, run.phi_q.b1, run.phi_q.w2, run.phi_q.b2, run.phi_q.relu, dev)
    pk = veda.Mlp(run.phi_k.w1, run.phi_k.b1, run.phi_k.w2, run.phi_k.b2, run.phi_k.relu, dev)
    rp1, ci1, _ = veda.veda_tile_score_select(run.plan, pq, pk, run.score_scale, k5, q_tiled=run.bufs["qt"],
                                              k_tiled=run.bufs["kt"], valid_mask=run.bufs["vm"])
    torch.cuda.synchronize()
    assert torch.equal(rp1, rp2) and torch.equal(ci1, ci2)
    rows = hz.sample_tiles(12240, 64, 5)
    s = run.bufs["s"][0].view(12240, 12240)[torch.as_tensor(rows, device=dev)].cpu().numpy()
    want = vo.select(s, 612)
    got = ci2.view(12240, 612)[torch.as_tensor(rows, device=dev)].cpu().numpy()
    assert np.array_equal(got, want)


# ---------------------------------------------------------------- supervision side
@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 64), ("f32", 128)])
def test_target_heatmap_and_recall(dtype, d):
    # full-attention target tile scores (max-pooled softmax) and Recall@k against the oracle:
    # ragged grid, odd tile counts, all three tile shapes, batch 2, then a subset of query tiles
    wl = wlm.custom_workload(f"heat_{dtype}_{d}", 4, d, dtype, (9, 18, 18), True, (25, 100), seed=61, batch=2)
    dev = torch.device("cuda:0")
    shapes = wlm.tile_shapes(wl)
    q, k, _ = wlm.make_qkv(wl, dev)
    plan = veda.Plan(wl.batch, wl.heads, wl.head_dim, wl.grid, shapes, wl.torch_dtype)
    qt, vm, _ = veda.veda_tile_layout(plan, q, veda.VEDA_TOKEN_MAJOR)
    kt, _, _ = veda.veda_tile_layout(plan, k, veda.VEDA_TOKEN_MAJOR, want_mask=False)
    scale = 1.0 / math.sqrt(d)
    heat = veda.veda_tile_heatmap(plan, qt, kt, vm, scale)
    torch.cuda.synchronize()
    rtol = 2e-4 if dtype == "bf16" else 2e-5
    refs = {}
    for b in range(wl.batch):
        for h in range(wl.heads):
            shape = tuple(int(x) for x in shapes[h])
            nt, soff = plan.tiles[h], plan.score_offset[h]
            ref = vo.tile_heatmap(hz.to_f32_numpy(q[b, h]), hz.to_f32_numpy(k[b, h]), wl.grid, shape, scale)
            got = heat[b, soff:soff + nt * nt].view(nt, nt).cpu().numpy().astype(np.float64)
            rel = np.abs(got - ref) / ref
            _say(f"[parity] {wl.name} b{b} h{h} {shape}: heat max rel err {rel.max():.2e}")
            assert rel.max() <= rtol, (b, h, rel.max())
            refs[(b, h)] = ref
    # a subset of query tiles: listed rows equal the full run, the others are not touched
    total = plan.total_tiles
    some = np.asarray(sorted({0, 1, total // 2, total - 1, plan.tile_offset[1] + 3}), np.int32)
    part = torch.full_like(heat, -7.0)
    veda.veda_tile_heatmap(plan, qt, kt, vm, scale, torch.as_tensor(some).to(dev), part)
    torch.cuda.synchronize()
    for h in range(wl.heads):
        nt, soff, toff = plan.tiles[h], plan.score_offset[h], plan.tile_offset[h]
        a = part[:, soff:soff + nt * nt].view(wl.batch, nt, nt)
        f = heat[:, soff:soff + nt * nt].view(wl.batch, nt, nt)
        listed = np.asarray([g - toff for g in some if toff <= g < toff + nt], np.int64)
        others = np.setdiff1d(np.arange(nt), listed)
        assert torch.equal(a[:, listed], f[:, listed]) and bool((a[:, others] == -7.0).all())
    # Recall@k of the estimator's selection against the selection from the target scores
    kph = wlm.keep_budget(wl, None, shapes)
    eq, ek = wlm.make_estimator(wl, "q"), wlm.make_estimator(wl, "k")
    s_est, _ = veda.veda_tile_score(plan, qt, kt, vm, veda.Mlp(eq.w1, eq.b1, eq.w2, eq.b2, eq.relu, dev),
                                    veda.Mlp(ek.w1, ek.b1, ek.w2, ek.b2, ek.relu, dev), hz.score_scale_of(wl))
    _, ci_est = veda.veda_tile_select(plan, s_est, kph)
    _, ci_tgt = veda.veda_tile_select(plan, heat, kph)
    rec = veda.veda_tile_recall(plan, kph, ci_est, ci_tgt)
    torch.cuda.synchronize()
    a_np, b_np = ci_est.cpu().numpy(), ci_tgt.cpu().numpy()
    nnz = int(sum(int(n) * int(kk) for n, kk in zip(plan.tiles, kph)))
    off = 0
    for h in range(wl.heads):
        nt, kk = plan.tiles[h], int(kph[h])
        for b in range(wl.batch):
            lo = b * nnz + off
            ref = vo.recall(a_np[lo:lo + nt * kk].reshape(nt, kk), b_np[lo:lo + nt * kk].reshape(nt, kk))
            assert abs(float(rec[b, h]) - ref) <= 1e-6, (b, h, float(rec[b, h]), ref)
        off += nt * kk
    same = veda.veda_tile_recall(plan, kph, ci_tgt, ci_tgt)
    assert bool((same == 1.0).all())


@pytest.mark.parametrize("dtype,d,tile_tokens", [("bf16", 128, 64), ("bf16", 64, 64), ("bf16", 128, 128), ("f32", 128, 64), ("f32", 64, 64)])
@pytest.mark.parametrize("grid", [(5, 9, 13), (17, 6, 7), (1, 5, 67), (9, 31, 33)])
def test_target_heatmap_at_edge_tiles(dtype, d, tile_tokens, grid):
    """Key tiles of every fill (half and empty steps), query tiles with fewer real rows than waves, more than 64
    key tiles for some heads (maxima go out 64 at a time), and listed tiles in no order, an odd number per head."""
    shapes = [(4, 4, 4), (1, 8, 8), (16, 2, 2), (64, 1, 1), (1, 1, 64)]
    shapes = np.asarray([(2 * a, b, c) for a, b, c in shapes] if tile_tokens == 128 else shapes, np.int32)
    wl = wlm.custom_workload("heat_edges", len(shapes), d, dtype, grid, False, (50, 100), seed=29)
    dev = torch.device("cuda:0")
    q, k, _ = wlm.make_qkv(wl, dev)
    plan = veda.Plan(1, wl.heads, d, grid, shapes, wl.torch_dtype, tile_tokens=tile_tokens)
    qt, vm, _ = veda.veda_tile_layout(plan, q, veda.VEDA_TOKEN_MAJOR)
    kt, _, _ = veda.veda_tile_layout(plan, k, veda.VEDA_TOKEN_MAJOR, want_mask=False)
    scale = 1.0 / math.sqrt(d)
    heat = veda.veda_tile_heatmap(plan, qt, kt, vm, scale)
    listed = torch.randperm(plan.total_tiles, generator=torch.Generator().manual_seed(1))[:plan.total_tiles // 2 | 1].to(torch.int32)
    part = veda.veda_tile_heatmap(plan, qt, kt, vm, scale, listed.to(dev), torch.full_like(heat, -7.0))
    kept, sums = veda.veda_tile_heatmap_rows(plan, qt, kt, vm, scale)
    again, _ = veda.veda_tile_heatmap_rows(plan, qt, kt, vm, scale, sums)
    torch.cuda.synchronize()
    for h in range(wl.heads):
        nt, soff, toff = plan.tiles[h], plan.score_offset[h], plan.tile_offset[h]
        ref = vo.tile_heatmap(hz.to_f32_numpy(q[0, h]), hz.to_f32_numpy(k[0, h]), grid, tuple(int(x) for x in shapes[h]), scale)
        got = heat[0, soff:soff + nt * nt].view(nt, nt)
        rel = np.abs(got.cpu().numpy().astype(np.float64) - ref) / ref
        assert rel.max() <= (2e-4 if dtype == "bf16" else 2e-5), (h, rel.max())
        # the rows' sums kept under this tiling and read under the same one: the same bits
        assert torch.equal(kept, heat) and torch.equal(again, heat)
        rows = [int(g) - toff for g in listed if toff <= int(g) < toff + nt]
        others = np.setdiff1d(np.arange(nt), rows)
        p = part[0, soff:soff + nt * nt].view(nt, nt)
        assert torch.equal(p[rows], got[rows]) and bool((p[others] == -7.0).all())


@pytest.mark.parametrize("dtype,d,tile_tokens", [("bf16", 128, 64), ("bf16", 64, 128), ("f32", 64, 64), ("f32", 128, 64)])
def test_row_sums_formed_under_another_tiling(dtype, d, tile_tokens):
    """What veda_tile_heatmap_rows is for: the sums written under one set of tile shapes, in token order, read under
    another (64- and 128-token tiles hand them to each other as well): scores against the oracle."""
    grid, batch = (9, 10, 14), 2
    first = np.asarray([[4, 4, 4], [1, 8, 8], [16, 2, 2]], np.int32)
    second = first[[1, 2, 0]] * np.asarray([tile_tokens // 64, 1, 1], np.int32)
    wl = wlm.custom_workload("cross", 3, d, dtype, grid, False, (50, 100), seed=41, batch=batch)
    q, k, _ = wlm.make_qkv(wl, torch.device("cuda:0"))
    scale, sums = 1.0 / math.sqrt(d), None
    for shapes, tokens in ((first, 64), (second, tile_tokens), (first, 64)):
        plan = veda.Plan(batch, 3, d, grid, shapes, wl.torch_dtype, tile_tokens=tokens)
        qt, vm, _ = veda.veda_tile_layout(plan, q)
        kt, _, _ = veda.veda_tile_layout(plan, k, want_mask=False)
        if sums is not None and tokens == 64 and shapes is first:      # and back: sums formed under the second set
            _, sums = veda.veda_tile_heatmap_rows(last[0], last[1], last[2], last[3], scale)
        heat, sums = veda.veda_tile_heatmap_rows(plan, qt, kt, vm, scale, sums)
        torch.cuda.synchronize()
        for b in range(batch):
            for h in range(3):
                nt, soff = plan.tiles[h], plan.score_offset[h]
                ref = vo.tile_heatmap(hz.to_f32_numpy(q[b, h]), hz.to_f32_numpy(k[b, h]), grid, tuple(int(x) for x in shapes[h]), scale)
                got = heat[b, soff:soff + nt * nt].view(nt, nt).cpu().numpy().astype(np.float64)
                rel = (np.abs(got - ref) / ref).max()
                assert rel <= (2e-4 if dtype == "bf16" else 2e-5), (tokens, b, h, rel)
        last = (plan, qt, kt, vm)


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 128), ("f32", 64)])
def test_target_scores_of_rows_whose_logits_rise_along_the_keys(dtype, d):
    """The softmax reference of a row moves many times after its first block, on both sides of the places where the
    running part of its denominator is put away (every 32 steps): logits rise by 60 over 80 key tiles, fall, or do neither,
    from row to row."""
    grid, n, rise = (4, 16, 80), 5120, 60.0
    g = torch.Generator().manual_seed(6)
    q, k = torch.randn((1, 1, n, d), generator=g), 0.5 * torch.randn((1, 1, n, d), generator=g)
    token = torch.arange(n)
    tile = (token // 80 % 16) // 4 * 20 + (token % 80) // 4                     # 4 x 20 tiles of 4x4x4
    q[0, 0, :, 0] = torch.tensor([1.0, -1.0, 0.0, 0.5])[token % 4]
    k[0, 0, :, 0] = (tile / 79.0 - 0.5) * rise * math.sqrt(d)
    q, k = (x.to(torch.bfloat16 if dtype == "bf16" else torch.float32).cuda() for x in (q, k))
    scale = 1.0 / math.sqrt(d)
    plan = veda.Plan(1, 1, d, grid, np.asarray([[4, 4, 4]], np.int32), q.dtype)
    qt, vm, _ = veda.veda_tile_layout(plan, q)
    kt, _, _ = veda.veda_tile_layout(plan, k, want_mask=False)
    heat, sums = veda.veda_tile_heatmap_rows(plan, qt, kt, vm, scale)
    again, _ = veda.veda_tile_heatmap_rows(plan, qt, kt, vm, scale, sums)
    torch.cuda.synchronize()
    assert torch.equal(again, heat)
    rows = np.arange(0, 80, 9)
    ref = vo.tile_heatmap(hz.to_f32_numpy(q[0, 0]), hz.to_f32_numpy(k[0, 0]), grid, (4, 4, 4), scale, query_tiles=rows)[rows]
    got = heat[0].view(80, 80)[torch.as_tensor(rows).cuda()].cpu().numpy().astype(np.float64)
    # a logit (and the row's reference) is a sum of d products rounded at the size of the sum, at most rise / 2 and the
    # noise beside it, then scaled; the denominator's sums have 16, 64 and 3 terms a lane, and moves beside them
    rtol = (2 * (d + 3) * (rise / 2 + 6.0) + 256) * 2.0 ** -24
    rel = np.abs(got - ref) / ref
    _say(f"[parity] rising logits {dtype} d {d}: max rel err {rel.max():.2e} of {rtol:.2e}, scores {ref.min():.1e} to {ref.max():.2f}")
    assert rel.max() <= rtol, rel.max()


@pytest.mark.parametrize("dtype,batch", [("bf16", 2), ("f32", 1)])
def test_listed_query_tiles_of_every_pattern(dtype, batch):
    """100 heads, lists on both sides of the window that pairs are looked for in (4096 entries), in order and not,
    the same even count in every head, single tiles: the listed rows as in the full run, the others untouched."""
    grid, heads, d = (8, 16, 24), 100, 64
    wl = wlm.custom_workload("lists", heads, d, dtype, grid, False, (50, 100), seed=37, batch=batch)
    q, k, _ = wlm.make_qkv(wl, torch.device("cuda:0"))
    plan = veda.Plan(batch, heads, d, grid, np.asarray([[4, 4, 4]] * heads, np.int32), wl.torch_dtype)
    qt, vm, _ = veda.veda_tile_layout(plan, q)
    kt, _, _ = veda.veda_tile_layout(plan, k, want_mask=False)
    heat = veda.veda_tile_heatmap(plan, qt, kt, vm, 0.125)
    n, total = plan.tiles[0], plan.total_tiles
    mixed = np.random.default_rng(9).permutation(total)
    lists = [np.arange(total), mixed, mixed[:4096], mixed[:4097], mixed[:257], np.arange(0, total, 2), np.arange(0, total, 12), np.arange(0, total, 24),
             np.concatenate([np.arange(i, total, n) for i in range(0, n, 3)]), np.asarray([total - 1]), np.asarray([n, n - 1, 1])]
    full = heat.view(batch, total, n)
    for listed in lists:
        listed = torch.as_tensor(listed.astype(np.int32)).cuda()
        part = veda.veda_tile_heatmap(plan, qt, kt, vm, 0.125, listed, torch.full_like(heat, -7.0)).view(batch, total, n)
        rest = torch.ones(total, dtype=torch.bool, device="cuda:0")
        rest[listed.long()] = False
        assert torch.equal(part[:, ~rest], full[:, ~rest]) and bool((part[:, rest] == -7.0).all()), len(listed)


@pytest.mark.parametrize("dtype,d,grid,shape", [
    ("bf16", 128, (5, 9, 13), (4, 4, 4)), ("bf16", 64, (9, 6, 10), (16, 2, 2)), ("f32", 128, (9, 6, 10), (16, 2, 2)), ("bf16", 128, (1, 1, 40), (1, 1, 64)),
    ("f32", 64, (5, 5, 17), (4, 4, 4)), ("bf16", 64, (21, 5, 7), (4, 4, 4))])
def test_target_scores_of_tiles_that_share_wavefronts(dtype, d, grid, shape):
    """Query tiles of few and of many real rows, packed into wavefronts together: any list of them gives the rows of a full run
    (a list packs them otherwise), with scratch and without; and with a mask that calls every slot real, which leaves fewer tiles to
    a workgroup than the geometry's, the rows of a tile are those of a call for that tile alone."""
    heads, dev, scale = 3, torch.device("cuda:0"), 1.0 / math.sqrt(d)
    wl = wlm.custom_workload("packed", heads, d, dtype, grid, False, (50, 100), seed=41, batch=2)
    q, k, _ = wlm.make_qkv(wl, dev)
    plan = veda.Plan(2, heads, d, grid, np.asarray([shape] * heads, np.int32), wl.torch_dtype)
    qt, vm, _ = veda.veda_tile_layout(plan, q)
    kt, _, _ = veda.veda_tile_layout(plan, k, want_mask=False)
    n, total = plan.tiles[0], plan.total_tiles
    lib, stream = veda.load(), torch.cuda.current_stream().cuda_stream
    rng = np.random.default_rng(5)
    for mask in (vm, torch.full_like(vm, -1)):
        full = veda.veda_tile_heatmap(plan, qt, kt, mask, scale).view(2, total, n)
        again = torch.empty_like(full)
        assert lib.veda_tile_heatmap(plan.handle, qt.data_ptr(), kt.data_ptr(), mask.data_ptr(), scale, None, 0, again.data_ptr(), stream) == veda.VEDA_OK
        assert torch.equal(full, again) and bool((full > 0).all())
        for count in sorted({1, min(2, total), min(5, total), (total + 1) // 2, total}):
            listed = torch.as_tensor(rng.permutation(total)[:count].astype(np.int32)).cuda()
            rest = torch.ones(total, dtype=torch.bool, device=dev)
            rest[listed.long()] = False
            part = veda.veda_tile_heatmap(plan, qt, kt, mask, scale, listed, torch.full_like(full, -7.0).view(2, -1)).view(2, total, n)
            assert torch.equal(part[:, ~rest], full[:, ~rest]) and bool((part[:, rest] == -7.0).all()), count
        if mask is vm:
            x, y = (t.view(2, heads, n * 64, d).double() for t in (qt, kt))
            real = ((vm.view(heads, n, 1) >> torch.arange(64, device=dev)) & 1).bool().view(1, heads, n * 64)
            s = torch.matmul(x, y.transpose(2, 3).contiguous()) * scale
            s = torch.softmax(s.masked_fill(~real[:, :, None], -math.inf), dim=3) * real[..., None]
            ref = s.view(2, heads, n, 64, n, 64).amax(dim=(3, 5)).view(2, total, n)
            assert ((full - ref).abs() <= (2e-4 if dtype == "bf16" else 2e-5) * ref).all()


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 128)])
@pytest.mark.parametrize("grid,shape", [((5, 9, 13), (4, 4, 4)), ((9, 6, 10), (16, 2, 2)), ((4, 8, 8), (4, 4, 4))])
def test_target_scores_where_query_rows_are_nan(dtype, d, grid, shape):
    """A row of NaN does not count for its tile, a tile of nothing else is NaN, full or not, and the others' scores are those of a call
    without, with scratch and without."""
    heads, scale = 2, 1.0 / math.sqrt(d)
    wl = wlm.custom_workload("nan_rows", heads, d, dtype, grid, False, (50, 100), seed=43)
    q, k, _ = wlm.make_qkv(wl, torch.device("cuda:0"))
    plan = veda.Plan(1, heads, d, grid, np.asarray([shape] * heads, np.int32), wl.torch_dtype)
    n, slots = plan.tiles[0], _tile_tokens(shape, grid)
    lib, stream, maps = veda.load(), torch.cuda.current_stream().cuda_stream, []
    kt, vm, _ = veda.veda_tile_layout(plan, k)
    for odd in (False, True):
        if odd:
            q[0, 0, slots[0, 0]] = math.nan
            for i in (1, n - 1):
                q[0, 0, slots[i][slots[i] >= 0]] = math.nan
        qt, _, _ = veda.veda_tile_layout(plan, q, want_mask=False)
        heat = veda.veda_tile_heatmap(plan, qt, kt, vm, scale).view(heads, n, n)
        again = torch.empty_like(heat)
        assert lib.veda_tile_heatmap(plan.handle, qt.data_ptr(), kt.data_ptr(), vm.data_ptr(), scale, None, 0, again.data_ptr(), stream) == veda.VEDA_OK
        torch.cuda.synchronize()
        assert torch.equal(heat.isnan(), again.isnan()) and torch.equal(heat.nan_to_num(7.0), again.nan_to_num(7.0))
        maps.append(heat)
    clean, odd = maps
    rest = torch.ones(heads, n, dtype=torch.bool, device="cuda:0")
    rest[0, [0, 1, n - 1]] = False
    assert torch.equal(odd[rest], clean[rest]) and bool(odd[0, [1, n - 1]].isnan().all()) and not bool(odd[0, 0].isnan().any())
    s = torch.softmax((q[0, 0, slots[0, 1:][slots[0, 1:] >= 0]].double() @ k[0, 0].double().T) * scale, dim=1).amax(dim=0)
    ref = torch.stack([s[t[t >= 0].cuda()].max() for t in slots])
    assert ((odd[0, 0] - ref).abs() <= (2e-4 if dtype == "bf16" else 2e-5) * ref).all()


@pytest.mark.parametrize("d", [64, 128])
def test_fp32_target_scores_below_the_smallest_normal_number(d):
    """Key tiles up to 102 below the row's maximum (natural units): their scores are subnormal, keep their order,
    and the top-k goes by it and not by the tile number."""
    grid, n, spread = (4, 16, 16), 1024, 102.0
    g = torch.Generator().manual_seed(5)
    q, k = torch.randn((1, 1, n, d), generator=g), 0.5 * torch.randn((1, 1, n, d), generator=g)
    q[..., 1:] *= 0.2
    q[..., 0] = 1.0
    token = torch.arange(n)
    tile = (token // 16 % 16) // 4 * 4 + (token % 16) // 4          # 4 x 4 tiles of 4x4x4
    k[0, 0, :, 0] = (tile - 15) / 15.0 * spread * math.sqrt(d)       # higher tile number, larger score
    scale = 1.0 / math.sqrt(d)
    plan = veda.Plan(1, 1, d, grid, np.asarray([[4, 4, 4]], np.int32), torch.float32)
    qt, vm, _ = veda.veda_tile_layout(plan, q.cuda())
    kt, _, _ = veda.veda_tile_layout(plan, k.cuda(), want_mask=False)
    heat = veda.veda_tile_heatmap(plan, qt, kt, vm, scale)
    kept, sums = veda.veda_tile_heatmap_rows(plan, qt, kt, vm, scale)
    again, _ = veda.veda_tile_heatmap_rows(plan, qt, kt, vm, scale, sums)
    _, ci = veda.veda_tile_select(plan, heat, [15])
    torch.cuda.synchronize()
    assert torch.equal(kept, heat) and torch.equal(again, heat)
    ref = vo.tile_heatmap(q[0, 0].numpy(), k[0, 0].numpy(), grid, (4, 4, 4), scale)
    assert ((ref > 0) & (ref < 2.0 ** -126)).sum() >= 32 and ref.min() < 2.0 ** -149
    # a logit is a sum of d products, each addition rounded at the size of the sum (at most the spread), then scaled and
    # taken from the reference; a score is rounded to a multiple of 2^-149 once
    rtol = (d + 3) * 2.0 ** -24 * (spread + 3.0)
    got = heat[0].view(16, 16).cpu().numpy().astype(np.float64)
    excess = (np.abs(got - ref) / (rtol * ref + 2.0 ** -149)).max()
    assert excess <= 1.0, (excess, int((got == 0.0).sum()))
    assert np.array_equal(ci.view(16, 15).cpu().numpy(), vo.select(ref.astype(np.float32), 15))


@pytest.mark.parametrize("dtype,d,tile_tokens,grid,heads", [
    ("bf16", 128, 64, (5, 30, 33), 5),       # tiles of every fill
    ("bf16", 64, 64, (8, 66, 64), 12),       # more work items than places in the scratch: 12 x 136 pairs and more
    ("bf16", 128, 128, (9, 31, 33), 5),      # halves without a token
    ("f32", 128, 64, (4, 62, 64), 15),       # more work items than places
    ("f32", 64, 64, (1, 5, 67), 5),
])
def test_heatmap_with_and_without_scratch(dtype, d, tile_tokens, grid, heads):
    _with_and_without_scratch(dtype, d, tile_tokens, grid, heads, 1)


@pytest.mark.parametrize("d", [64, 128])
def test_heatmap_of_whole_tiles_with_more_items_than_places(d):
    """128-token tiles, all 6720 and 5042 listed ones of two samples: more than the 1024 or 1280 places, so that a workgroup goes on
    with its scratch and its LDS as the tile before left them."""
    _with_and_without_scratch("bf16", d, 128, (8, 66, 64), 12, 2)


def _with_and_without_scratch(dtype, d, tile_tokens, grid, heads, batch):
    """The logits formed once (with scratch) or twice: the same bits, all rows and listed ones, with rows and keys that
    are not finite among them, and nothing outside the scratch is touched."""
    shapes = [(4, 4, 4), (1, 8, 8), (16, 2, 2), (64, 1, 1), (1, 1, 64)]
    shapes = [(2 * a, b, c) for a, b, c in shapes] if tile_tokens == 128 else shapes
    shapes = np.asarray([shapes[h % 5] for h in range(heads)] if heads < 12 else [shapes[h % 2] for h in range(heads)], np.int32)
    wl = wlm.custom_workload("one_walk", heads, d, dtype, grid, False, (50, 100), seed=37, batch=batch)
    dev = torch.device("cuda:0")
    q, k, _ = wlm.make_qkv(wl, dev)
    n_tok = q.shape[2]
    q[0, 0, 3] = float("nan")
    q[0, 1, :n_tok // 2] = float("inf")
    k[0, 2, 5] = float("-inf")
    k[0, 3, n_tok // 3:n_tok // 2] = float("nan")
    plan = veda.Plan(batch, heads, d, grid, shapes, wl.torch_dtype, tile_tokens=tile_tokens)
    qt, vm, _ = veda.veda_tile_layout(plan, q, veda.VEDA_TOKEN_MAJOR)
    kt, _, _ = veda.veda_tile_layout(plan, k, veda.VEDA_TOKEN_MAJOR, want_mask=False)
    lib, scale, stream = veda.load(), 1.0 / math.sqrt(d), torch.cuda.current_stream().cuda_stream
    listed = torch.randperm(plan.total_tiles, generator=torch.Generator().manual_seed(2))[:plan.total_tiles * 3 // 4 | 1]
    for rows in (None, listed.to(torch.int32).to(dev)):
        n = 0 if rows is None else rows.numel()
        ptr = None if rows is None else rows.data_ptr()
        heats = [torch.full((batch, plan.score_elems), -7.0, device=dev) for _ in range(3)]
        need = int(lib.veda_plan_heatmap_workspace_bytes(plan.handle, n))
        around = torch.full((need + 512,), 77, dtype=torch.uint8, device=dev)
        args = (plan.handle, qt.data_ptr(), kt.data_ptr(), vm.data_ptr(), scale, ptr, n)
        ws = around.data_ptr() + 256
        assert lib.veda_tile_heatmap(*args, heats[0].data_ptr(), stream) == veda.VEDA_OK
        assert lib.veda_tile_heatmap_ws(*args, None, heats[1].data_ptr(), ws, need - 1, stream) == veda.VEDA_ERR_WORKSPACE
        assert lib.veda_tile_heatmap_ws(*args, None, heats[1].data_ptr(), ws, need, stream) == veda.VEDA_OK
        veda.veda_tile_heatmap(plan, qt, kt, vm, scale, rows, heats[2])
        torch.cuda.synchronize()
        assert bool((around[:256] == 77).all()) and bool((around[-256:] == 77).all())
        assert torch.equal(heats[0].view(torch.int32), heats[1].view(torch.int32))
        assert torch.equal(heats[0].view(torch.int32), heats[2].view(torch.int32))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("where,value", [("k", -math.inf), ("k", math.inf), ("k", math.nan), ("k", 3.4e38), ("q", -math.inf),
                                         ("v", math.inf), ("v", math.nan), ("v", 3.4e38), ("q", 1e-30), ("v", 1e-35)])
def test_fp32_kernels_on_numbers_a_split_does_not_hold(d, where, value):
    """Numbers that do not survive the split into bf16 parts (not finite, or rounded to infinity) or whose parts are
    subnormal: outputs and target scores are those of the formulas, not finite exactly where those are not."""
    grid, heads = (4, 9, 22), 2
    wl = wlm.custom_workload("odd_numbers", heads, d, "f32", grid, False, (50, 100), seed=43)
    dev = torch.device("cuda:0")
    q, k, v = wlm.make_qkv(wl, dev)
    x = {"q": q, "k": k, "v": v}[where]
    if abs(value) < 1.0:
        x *= value
    else:
        x[0, 0, 100, 5] = value   # head 1 stays as it is
        x[0, 0, 333, d - 1] = value
    shape = (4, 4, 4)
    plan = veda.Plan(1, heads, d, grid, np.asarray([shape] * heads, np.int32), torch.float32)
    qt, vm, _ = veda.veda_tile_layout(plan, q)
    kt, _, _ = veda.veda_tile_layout(plan, k, want_mask=False)
    vt, _, _ = veda.veda_tile_layout(plan, v, veda.VEDA_CHANNEL_MAJOR, want_mask=False)
    n, scale = plan.tiles[0], 1.0 / math.sqrt(d)
    keep = torch.rand((heads * n, n), generator=torch.Generator().manual_seed(3)).argsort(dim=1)[:, :n // 2].sort(dim=1)[0]
    rp = (torch.arange(heads * n + 1, dtype=torch.int32) * (n // 2)).to(dev)
    out, _ = veda.veda_sparse_attn_fwd(plan, qt, kt, vt, vm, rp, keep.reshape(-1).to(torch.int32).to(dev), scale)
    heat = veda.veda_tile_heatmap(plan, qt, kt, vm, scale).cpu().view(heads, n, n)
    kept, sums = veda.veda_tile_heatmap_rows(plan, qt, kt, vm, scale)
    again, _ = veda.veda_tile_heatmap_rows(plan, qt, kt, vm, scale, sums)
    assert torch.equal(kept.cpu().view(heads, n, n).nan_to_num(-1.0), heat.nan_to_num(-1.0))
    assert torch.equal(again.cpu().view(heads, n, n).nan_to_num(-1.0), heat.nan_to_num(-1.0))
    out, q, k, v = (t[0].cpu() for t in (out, q, k, v))
    slots = _tile_tokens(shape, grid)
    for h in range(heads):
        # logits as fp32 has them (a product of finite numbers may leave its range; the attention scales the queries, the
        # target scores the products), the rest in 64 bits
        log2e = 1.4426950408889634
        s = ((q[h].double() * (scale * log2e)) @ k[h].double().T).float().double() / log2e
        full = torch.softmax((q[h].double() @ k[h].double().T).float().double() * scale, dim=1)
        for i in range(n):
            rows = slots[i][slots[i] >= 0]
            cols = slots[keep[h * n + i]].reshape(-1)
            cols = cols[cols >= 0]
            p = torch.softmax(s[rows][:, cols], dim=1)
            ref = p @ v[h][cols].double()
            got = out[h][rows].double()
            assert torch.equal(torch.isfinite(got), torch.isfinite(ref.float())), (h, i)
            ok = torch.isfinite(ref.float())
            # a sum of up to 384 products, each with a weight off by the error of its logit, itself a sum of d: below
            # (384 + 2 * 8 * d) * 2^-24 of the sum of |p v| for logits up to 8, and half a subnormal for each
            bound = 2.0 ** -24 * (384 + 16 * d) * (p @ v[h][cols].double().abs()) + 384 * 2.0 ** -150
            assert ((got - ref).abs() <= bound)[ok].all(), (h, i)
            block = torch.stack([full[rows][:, t[t >= 0]].nan_to_num(-1.0).amax() for t in slots])
            if torch.isfinite(full[rows]).all():
                assert ((heat[h, i] - block).abs() <= 2e-5 * block + 1e-30).all(), (h, i)


@pytest.mark.parametrize("dtype,d,tile_tokens,all_tiles,listed", [
    ("bf16", 128, 64, 4, 4), ("bf16", 128, 128, 4, 4), ("bf16", 64, 64, 5, 4), ("bf16", 64, 128, 5, 5), ("f32", 128, 64, 2, 2), ("f32", 64, 64, 3, 3)])
def test_heatmap_scratch_is_that_of_the_resident_workgroups(dtype, d, tile_tokens, all_tiles, listed):
    """Workgroups on a compute unit as hipOccupancyMaxActiveBlocksPerMultiprocessor gives them (fp32, d = 64: one fewer), 256
    compute units."""
    shape = (4, 4, tile_tokens // 16)
    plan = veda.Plan(3, 40, d, (20, 20, 400), np.asarray([shape] * 40, np.int32), torch.bfloat16 if dtype == "bf16" else torch.float32, tile_tokens=tile_tokens)
    halves = plan.tiles[0] * tile_tokens // 64
    need = veda.load().veda_plan_heatmap_workspace_bytes
    assert need(plan.handle, 0) == 512 + 512 * halves * 256 * all_tiles
    assert need(plan.handle, plan.total_tiles) == 512 + 512 * halves * 256 * listed
    assert need(plan.handle, 16) <= 512 + 512 * halves * 64


@pytest.mark.parametrize("tiles,places,bounded", [(3840, 1024, False), (4352, 960, False), (8256, 512, True)])
def test_heatmap_scratch_has_an_upper_bound(tiles, places, bounded):
    """Heads whose scratch would pass 2 GiB get by with fewer places, and from half of them on with none, with the same bits."""
    grid, dev = (16, 4 * 16, 4 * (tiles // 64)), torch.device("cuda:0")
    wl = wlm.custom_workload("large_heads", 1, 128, "bf16", grid, False, (50, 100), seed=67)
    q, k, _ = wlm.make_qkv(wl, dev)
    plan = veda.Plan(1, 1, 128, grid, np.asarray([(4, 4, 4)], np.int32), torch.bfloat16)
    assert plan.total_tiles == tiles
    qt, vm, _ = veda.veda_tile_layout(plan, q)
    kt, _, _ = veda.veda_tile_layout(plan, k, want_mask=False)
    heats = [torch.empty((1, plan.score_elems), device=dev) for _ in range(3)]
    need = int(veda.load().veda_plan_heatmap_workspace_bytes(plan.handle, 0))
    assert need == 512 + 512 * tiles * places and (need > veda.HEATMAP_SCRATCH_BYTES) == bounded
    scale, stream = 1.0 / math.sqrt(128), torch.cuda.current_stream().cuda_stream

    def grows(f):
        torch.cuda.empty_cache()
        torch.cuda.reset_peak_memory_stats()
        before = torch.cuda.memory_allocated()
        r = f()
        torch.cuda.synchronize()
        return r, torch.cuda.max_memory_allocated() - before

    _, used = grows(lambda: veda.veda_tile_heatmap(plan, qt, kt, vm, scale, None, heats[0]))
    assert used == 0 if bounded else used >= need
    (heat, sums), used = grows(lambda: veda.veda_tile_heatmap_rows(plan, qt, kt, vm, scale))
    assert used - (heat.numel() + sums.numel()) * 4 < (2 ** 20 if bounded else need + 2 ** 22)
    ws = torch.empty(need, dtype=torch.uint8, device=dev)
    assert veda.load().veda_tile_heatmap_ws(plan.handle, qt.data_ptr(), kt.data_ptr(), vm.data_ptr(), scale, None, 0, None,
                                            heats[1].data_ptr(), ws.data_ptr(), need, stream) == veda.VEDA_OK
    assert veda.load().veda_tile_heatmap(plan.handle, qt.data_ptr(), kt.data_ptr(), vm.data_ptr(), scale, None, 0, heats[2].data_ptr(),
                                         stream) == veda.VEDA_OK
    assert torch.equal(heats[0], heats[1]) and torch.equal(heats[0], heats[2]) and torch.equal(heats[0], heat)


def test_heatmap_refuses_lists_longer_than_the_tiles():
    """As an invalid argument, with and without scratch: no scratch is said to be needed for them."""
    plan = veda.Plan(1, 1, 64, (4, 4, 16), np.asarray([(4, 4, 4)], np.int32), torch.bfloat16)
    x, vm = torch.zeros((1, 4, 64 * 64), dtype=torch.bfloat16, device="cuda"), torch.full((4,), -1, dtype=torch.int64, device="cuda")
    listed = torch.arange(5, dtype=torch.int32, device="cuda") % 4
    heat = torch.empty((1, 16), device="cuda")
    for call in (lambda: veda.veda_tile_heatmap(plan, x, x, vm, 0.125, listed, heat),
                 lambda: veda._check(veda.load().veda_tile_heatmap(plan.handle, x.data_ptr(), x.data_ptr(), vm.data_ptr(), 0.125, listed.data_ptr(), 5,
                                                                   heat.data_ptr(), None), "veda_tile_heatmap")):
        with pytest.raises(veda.VedaError) as e:
            call()
        assert e.value.status == veda.VEDA_ERR_INVALID_ARG


def test_heatmap_of_many_small_samples():
    """128 heads of one tile: eight workgroups for each (every head's pair falls to the first die), so that 16384 samples are
    2^24 of them, more than a grid's first dimension takes."""
    heads, batch, dev = 128, 16384, torch.device("cuda:0")
    plan = veda.Plan(batch, heads, 64, (4, 4, 4), np.asarray([(4, 4, 4)] * heads, np.int32), torch.bfloat16)
    x = torch.zeros((batch, heads, 64 * 64), dtype=torch.bfloat16, device=dev)
    for b in (0, 1, batch // 2, batch - 1):
        x[b] = torch.randn((heads, 64 * 64), device=dev, generator=torch.Generator(device=dev).manual_seed(b)).bfloat16()
    vm = torch.full((heads,), -1, dtype=torch.int64, device=dev)
    heat = torch.full((batch, heads), -7.0, device=dev)
    stream = torch.cuda.current_stream().cuda_stream
    assert veda.load().veda_tile_heatmap(plan.handle, x.data_ptr(), x.data_ptr(), vm.data_ptr(), 0.125, None, 0, heat.data_ptr(),
                                         stream) == veda.VEDA_OK
    assert torch.equal(heat, veda.veda_tile_heatmap(plan, x, x, vm, 0.125))
    assert bool((heat[2] == 1.0 / 64).all())
    for b in (0, 1, batch // 2, batch - 1):
        t = x[b].view(heads, 64, 64).float()
        ref = torch.softmax(torch.bmm(t, t.transpose(1, 2).contiguous()) * 0.125, dim=2).amax(dim=(1, 2))
        assert ((heat[b] - ref).abs() <= 1e-5 * ref).all()


def _tile_tokens(shape, grid):
    """Token of every slot of every tile, -1 for padding: [tiles, 64]."""
    ax = [torch.where(torch.arange(-(-n // e) * e) < n, torch.arange(-(-n // e) * e), -10 ** 6).view(-1, e) for e, n in zip(shape, grid)]
    t = (ax[0][:, None, None, :, None, None] * grid[1] + ax[1][None, :, None, None, :, None]) * grid[2] + ax[2][None, None, :, None, None, :]
    return t.clamp(min=-1).reshape(-1, shape[0] * shape[1] * shape[2])


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("qs,ks,vs,gap,same", [
    (1.0, 1.0, 1e-34, False, True), (1.0, 1.0, 1e-35, False, True), (1.0, 1.0, 1e-37, False, True), (1.0, 1.0, 1e-41, False, True),
    (1e-36, 1e36, 1.0, False, False), (1e-33, 1e33, 1.0, False, False), (1e36, 1e-36, 1.0, False, True), (1e10, 1e-10, 1.0, False, False),
    (1.0, 1.0, 1.0, True, True), (1.0, 1.0, 1e12, True, True),
    (1.0, 1.0, 1e-3, False, False), (1.0, 1.0, 1e3, False, False),
])
def test_fp32_splits_lose_nothing_of_small_numbers(d, qs, ks, vs, gap, same):
    """Operands and probabilities with parts below what bf16 holds (2^-133), and ordinary ones beside them: the split products
    are no further from 64 bits than the fp32 ones, and where they cannot say so the result is that of the fp32 ones."""
    grid, n = (4, 4, 72), 18
    wl = wlm.custom_workload("small_numbers", 1, d, "f32", grid, False, (50, 100), seed=61)
    q, k, v = wlm.make_qkv(wl, torch.device("cuda:0"))
    q *= qs
    k *= ks
    v *= vs
    if gap:   # all weight on one key without a value, the others' weights around 2^-121
        k *= 0.01
        q[..., 0], k[..., 0] = math.sqrt(d), 0.0
        k[0, 0, 7, 0], v[0, 0, 7] = 84.0, 0.0
    plan = veda.Plan(1, 1, d, grid, np.asarray([(4, 4, 4)], np.int32), torch.float32)
    qt, vm, _ = veda.veda_tile_layout(plan, q)
    kt, _, _ = veda.veda_tile_layout(plan, k, want_mask=False)
    vt, _, _ = veda.veda_tile_layout(plan, v, veda.VEDA_CHANNEL_MAJOR, want_mask=False)
    rp = torch.arange(n + 1, dtype=torch.int32, device="cuda") * n
    ci = torch.arange(n, dtype=torch.int32, device="cuda").repeat(n)
    scale, outs = 1.0 / math.sqrt(d), {}
    for form in (veda.VEDA_PRODUCTS_FP32, 0, veda.VEDA_PRODUCTS_SPLIT):
        plan.set_option(veda.VEDA_OPT_FP32_PRODUCTS, form)
        outs[form] = [t[0, 0].cpu() for t in veda.veda_sparse_attn_fwd(plan, qt, kt, vt, vm, rp, ci, scale, want_lse=True)]
    s = (q[0, 0].double() @ k[0, 0].double().T).cpu() * scale
    ref = torch.softmax(s, dim=1) @ v[0, 0].cpu().double()
    err = {f: ((o.double() - ref).norm() / ref.norm()).item() for f, (o, _) in outs.items()}
    _say(f"[parity] fp32 products d {d} q {qs} k {ks} v {vs} gap {gap}: from 64 bits {err}")
    for form in (0, veda.VEDA_PRODUCTS_SPLIT):
        assert err[form] <= err[veda.VEDA_PRODUCTS_FP32]
        assert torch.equal(outs[form][0], outs[veda.VEDA_PRODUCTS_FP32][0]) == same
        assert (outs[form][1].double() - torch.logsumexp(s, dim=1)).abs().max() <= 1e-5 * max(1.0, s.abs().max().item())


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("walk", [0, 1])
def test_fp32_second_walk_after_a_long_first(d, walk):
    """Work items whose unions outgrow the step table's ring (256 entries), walked again for numbers that are not finite: the bits of
    VEDA_PRODUCTS_FP32, and for the others those of the same call without such numbers."""
    n = 400
    grid = (4, 4, 4 * n)
    wl = wlm.custom_workload("again", 1, d, "f32", grid, False, (50, 100), seed=71)
    q, k, v = wlm.make_qkv(wl, torch.device("cuda:0"))
    plan = veda.Plan(1, 1, d, grid, np.asarray([(4, 4, 4)], np.int32), torch.float32)
    plan.set_option(veda.VEDA_OPT_ATTN_LIST_WALK, walk)
    g = torch.Generator().manual_seed(6)
    keep = torch.stack([torch.randperm(n, generator=g)[:200].sort()[0] for _ in range(n)])
    for i in range(0, n, 2):
        assert len(set(keep[i].tolist()) | set(keep[i + 1].tolist())) > 256
    rp = (torch.arange(n + 1, dtype=torch.int32) * 200).cuda()
    ci = keep.reshape(-1).to(torch.int32).cuda()
    slots = _tile_tokens((4, 4, 4), grid)
    hit = (keep == 390).any(dim=1)   # the tile of the infinity in V, kept late in the walk
    hit[37] = True                   # and the one of the NaN in Q
    hit = hit.view(-1, 2).any(dim=1).repeat_interleave(2)
    assert 0 < int(hit.sum()) < n
    outs = []
    for odd, form in ((False, veda.VEDA_PRODUCTS_SPLIT), (True, veda.VEDA_PRODUCTS_SPLIT), (True, veda.VEDA_PRODUCTS_FP32)):
        if odd:
            v[0, 0, slots[390, 5], 3] = math.inf
            q[0, 0, slots[37, 63], 0] = math.nan
        plan.set_option(veda.VEDA_OPT_FP32_PRODUCTS, form)
        qt, vm, _ = veda.veda_tile_layout(plan, q)
        kt, _, _ = veda.veda_tile_layout(plan, k, want_mask=False)
        vt, _, _ = veda.veda_tile_layout(plan, v, veda.VEDA_CHANNEL_MAJOR, want_mask=False)
        outs.append(veda.veda_sparse_attn_fwd(plan, qt, kt, vt, vm, rp, ci, 1.0 / math.sqrt(d))[0][0, 0].cpu()[slots])
    clean, again, chains = outs
    assert torch.equal(again[~hit], clean[~hit]) and not torch.equal(chains[~hit], clean[~hit])
    assert torch.equal(again[hit].isnan(), chains[hit].isnan()) and torch.equal(again[hit].nan_to_num(7.0), chains[hit].nan_to_num(7.0))
    assert bool(again[hit].isinf().any()) and bool(again[37, 63].isnan().all())


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("recipe", ["unit", "amp"])
@pytest.mark.parametrize("kept", [16, 63, 192, 193, 400])
def test_fp32_products_against_64_bits(d, recipe, kept):
    """The split products are nearer to 64 bits than the fp32 ones at every length and at larger logits ("amp"), and the default form
    stays within the fp32 bar, 1e-4 of the outputs' root mean square, of the fp32 ones (seen: up to 5.8e-5, after 192 tiles)."""
    n = 400
    grid = (4, 4, 4 * n)
    wl = wlm.custom_workload("nearness", 1, d, "f32", grid, False, (50, 100), seed=73, recipe=recipe)
    q, k, v = wlm.make_qkv(wl, torch.device("cuda:0"))
    plan = veda.Plan(1, 1, d, grid, np.asarray([(4, 4, 4)], np.int32), torch.float32)
    qt, vm, _ = veda.veda_tile_layout(plan, q)
    kt, _, _ = veda.veda_tile_layout(plan, k, want_mask=False)
    vt, _, _ = veda.veda_tile_layout(plan, v, veda.VEDA_CHANNEL_MAJOR, want_mask=False)
    keep = torch.rand((n, n), generator=torch.Generator().manual_seed(7)).argsort(dim=1)[:, :kept].sort(dim=1)[0]
    rp = (torch.arange(n + 1, dtype=torch.int32) * kept).cuda()
    ci, scale, outs = keep.reshape(-1).to(torch.int32).cuda(), 1.0 / math.sqrt(d), {}
    slots = _tile_tokens((4, 4, 4), grid)
    for form in (0, veda.VEDA_PRODUCTS_FP32, veda.VEDA_PRODUCTS_SPLIT):
        plan.set_option(veda.VEDA_OPT_FP32_PRODUCTS, form)
        outs[form] = veda.veda_sparse_attn_fwd(plan, qt, kt, vt, vm, rp, ci, scale)[0][0, 0][slots.cuda()].double()
    assert torch.equal(outs[0], outs[veda.VEDA_PRODUCTS_SPLIT if kept <= 192 else veda.VEDA_PRODUCTS_FP32])
    ref = torch.empty_like(outs[0])
    order = slots.cuda()
    q64, k64, v64 = q[0, 0].double(), k[0, 0].double(), v[0, 0].double()
    for i in range(n):
        cols = order[keep[i].cuda()].reshape(-1)
        ref[i] = torch.softmax((q64[order[i]] @ k64[cols].T) * scale, dim=1) @ v64[cols]
    err = {f: ((o - ref).norm() / ref.norm()).item() for f, o in outs.items()}
    apart = ((outs[0] - outs[veda.VEDA_PRODUCTS_FP32]).abs().max() / ref.square().mean().sqrt()).item()
    _say(f"[parity] fp32 products d {d} {recipe} kept {kept}: from 64 bits {err}, the default and the fp32 form apart by {apart:.2e}")
    assert err[veda.VEDA_PRODUCTS_SPLIT] < err[veda.VEDA_PRODUCTS_FP32]
    assert apart <= 1e-4


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("walk", [0, 1])
def test_fp32_products_by_list_length(d, walk):
    """Lists on both sides of the length at which the split products end, in one call: the rows of short lists have the
    bits of VEDA_PRODUCTS_SPLIT, those of pairs with a longer one the bits of VEDA_PRODUCTS_FP32, and all lie within the fp32
    bar of the formulas."""
    grid, heads, n = (4, 4, 4 * 231), 1, 231
    wl = wlm.custom_workload("lengths", heads, d, "f32", grid, False, (50, 100), seed=53)
    dev = torch.device("cuda:0")
    q, k, v = wlm.make_qkv(wl, dev)
    plan = veda.Plan(1, heads, d, grid, np.asarray([(4, 4, 4)], np.int32), torch.float32)
    plan.set_option(veda.VEDA_OPT_ATTN_LIST_WALK, walk)
    qt, vm, _ = veda.veda_tile_layout(plan, q)
    kt, _, _ = veda.veda_tile_layout(plan, k, want_mask=False)
    vt, _, _ = veda.veda_tile_layout(plan, v, veda.VEDA_CHANNEL_MAJOR, want_mask=False)
    g = torch.Generator().manual_seed(5)
    lengths = [(1, 2, 63, 64, 129, 191, 192, 193, 194, 230, 231)[i % 11] for i in range(n)]
    lists = [torch.randperm(n, generator=g)[:m].sort()[0] for m in lengths]
    rp = torch.tensor([0] + list(np.cumsum(lengths)), dtype=torch.int32, device=dev)
    ci = torch.cat(lists).to(torch.int32).to(dev)
    outs = {}
    for option in (0, veda.VEDA_PRODUCTS_FP32, veda.VEDA_PRODUCTS_SPLIT):
        plan.set_option(veda.VEDA_OPT_FP32_PRODUCTS, option)
        outs[option], _ = veda.veda_sparse_attn_fwd(plan, qt, kt, vt, vm, rp, ci, 1.0 / math.sqrt(d))
        outs[option] = outs[option][0, 0].cpu()
    with pytest.raises(veda.VedaError):
        plan.set_option(veda.VEDA_OPT_FP32_PRODUCTS, 3)
    slots = _tile_tokens((4, 4, 4), grid)
    s = (q[0, 0].double() @ k[0, 0].double().T).cpu() / math.sqrt(d)
    assert not torch.equal(outs[1], outs[2])
    for i in range(n):
        pair = [j for j in (i, i ^ 1) if j < n]   # tiles of a row of tiles pair up along it
        want = 1 if max(lengths[j] for j in pair) > 192 else 2
        assert torch.equal(outs[0][slots[i]], outs[want][slots[i]]), (i, lengths[i])
        cols = slots[lists[i]].reshape(-1)
        ref = torch.softmax(s[slots[i]][:, cols], dim=1) @ v[0, 0].cpu()[cols].double()
        for option in (1, 2):
            assert (outs[option][slots[i]].double() - ref).abs().max() <= 1e-4


def _fp32_forms(d, heads, batch, grid, shape, lengths, odd, walk):
    """Outputs of one call in both orders of the steps, or of its first sample in calls of several sizes."""
    dev, n = torch.device("cuda:0"), int(np.prod([-(-g // s) for g, s in zip(grid, shape)]))
    wl = wlm.custom_workload("forms", heads, d, "f32", grid, False, (50, 100), seed=83)
    q, k, v = wlm.make_qkv(wl, dev)
    if odd:   # in the first head, some of whose tiles keep them
        v[0, 0, -1, 3], q[0, 0, 5, 0] = math.inf, math.nan
        v[0, 0, 7] *= 1e-30
    plan = veda.Plan(batch, heads, d, grid, np.asarray([shape] * heads, np.int32), torch.float32)
    plan.set_option(veda.VEDA_OPT_ATTN_LIST_WALK, walk)
    qt, vm, _ = veda.veda_tile_layout(plan, q.expand(batch, -1, -1, -1).contiguous())
    kt, _, _ = veda.veda_tile_layout(plan, k.expand(batch, -1, -1, -1).contiguous(), want_mask=False)
    vt, _, _ = veda.veda_tile_layout(plan, v.expand(batch, -1, -1, -1).contiguous(), veda.VEDA_CHANNEL_MAJOR, want_mask=False)
    rng = np.random.default_rng(9)
    lists = [np.sort(rng.choice(n, lengths[rng.integers(len(lengths))], replace=False)) for _ in range(heads * n)] * batch
    rp = torch.as_tensor(np.concatenate([[0], np.cumsum([len(x) for x in lists])]).astype(np.int32)).to(dev)
    ci = torch.as_tensor(np.concatenate(lists).astype(np.int32)).to(dev)
    out, lse = veda.veda_sparse_attn_fwd(plan, qt, kt, vt, vm, rp, ci, 1.0 / math.sqrt(d), want_lse=True)
    torch.cuda.synchronize()
    assert (not odd) or bool(out[0, 0].isnan().any()) and not bool(out[0, 0].isnan().all())
    return out[0].nan_to_num(7.0, 8.0, 9.0).cpu(), lse[0].nan_to_num(7.0, 8.0, 9.0).cpu()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("heads", [1, 6])
@pytest.mark.parametrize("odd", [False, True])
def test_fp32_forms_are_the_same_in_both_orders(d, heads, odd):
    """Ragged grids with lists on both sides of the length at which the split products end, and numbers that are formed again (an
    infinity, a NaN, values too small for their parts): the rows' bits do not depend on how the steps are found."""
    table, walked = (_fp32_forms(d, heads, 1, (9, 33, 33), (4, 4, 4), (1, 20, 191, 192, 193, 240), odd, walk) for walk in (0, 1))
    assert torch.equal(table[0], walked[0]) and torch.equal(table[1], walked[1])


@pytest.mark.parametrize("d", [64, 128])
def test_fp32_forms_of_a_sample_alone_and_in_a_batch(d):
    """Heads whose lists are all short, with numbers that are formed again: a tile's form is its own, in calls of one
    tile to a workgroup, of pairs and of thin tiles in fours, and in either order of the steps."""
    first = _fp32_forms(d, 2, 1, (5, 9, 45), (4, 4, 4), (1, 3, 20), True, 0)
    for batch in (1, 4, 5, 20):
        for walk in (0, 1):
            got = _fp32_forms(d, 2, batch, (5, 9, 45), (4, 4, 4), (1, 3, 20), True, walk)
            assert torch.equal(got[0], first[0]) and torch.equal(got[1], first[1]), (batch, walk)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_row_sums_have_no_place_for_padded_slots(dtype):
    """A mask that calls padded slots real: their rows have no token, so no sums are kept for them (what lies around
    the buffer stays as it was) and they take no part in the scores.  The padded keys count, as zeros."""
    grid, d, heads, shape = (3, 5, 7), 64, 3, (4, 4, 4)
    wl = wlm.custom_workload("all_ones", heads, d, dtype, grid, False, (50, 100), seed=31)
    q, k, _ = wlm.make_qkv(wl, torch.device("cuda:0"))
    plan = veda.Plan(1, heads, d, grid, np.asarray([shape] * heads, np.int32), wl.torch_dtype)
    qt, vm, _ = veda.veda_tile_layout(plan, q)
    kt, _, _ = veda.veda_tile_layout(plan, k, want_mask=False)
    ones = torch.full_like(vm, -1)
    around = torch.full((heads * plan.tokens + 128, 2), -7.0, device="cuda:0")
    sums = around[64:64 + heads * plan.tokens].view(1, heads, plan.tokens, 2)
    lib, scale, heat = veda.load(), 1.0 / math.sqrt(d), torch.empty((1, plan.score_elems), device="cuda:0")
    maps = []
    for have in (0, 1):
        assert lib.veda_tile_heatmap_rows(plan.handle, qt.data_ptr(), kt.data_ptr(), ones.data_ptr(), scale, sums.data_ptr(), have,
                                          heat.data_ptr(), torch.cuda.current_stream().cuda_stream) == veda.VEDA_OK
        torch.cuda.synchronize()
        maps.append(heat.clone())
    assert torch.equal(maps[0], maps[1])
    assert bool((around[:64] == -7.0).all()) and bool((around[-64:] == -7.0).all()) and bool((sums[..., 1] > 0).all())
    n = plan.tiles[0]
    real = ((vm.view(heads, n, 1) >> torch.arange(64, device=vm.device)) & 1).bool()
    s = torch.matmul(qt.view(heads, n * 64, d).float(), kt.view(heads, n * 64, d).float().transpose(1, 2).contiguous()) * scale
    ref = (torch.softmax(s.double(), dim=2) * real.view(heads, -1, 1)).view(heads, n, 64, n, 64).amax(dim=(2, 4))
    assert ((maps[0].view(heads, n, n) - ref).abs() / ref).max() <= (2e-4 if dtype == "bf16" else 2e-5)


@pytest.mark.parametrize("grid,k", [((4, 8, 8), 1), ((4, 8, 8), 4), ((9, 36, 36), 65), ((9, 36, 36), 243), ((8, 364, 368), 130)])
def test_recall_of_constructed_lists(grid, k):
    """Lists in any order, one to several passes of a wavefront over them, whole rows, entries that are no tile
    (all pairs are compared then: equal entries count whatever they are), and rows longer than the bitmap."""
    shapes = np.asarray([[4, 4, 4], [1, 8, 8]], np.int32)
    plan = veda.Plan(1, 2, 64, grid, shapes, torch.float32)
    rng = np.random.default_rng(k)
    ks = [min(k, n) for n in plan.tiles]
    lists, ref = [[], []], []
    for n, kk in zip(plan.tiles, ks):
        m = n
        a = np.argsort(rng.random((m, min(n, 4 * kk))), axis=1)[:, :kk].astype(np.int32)
        b = np.argsort(rng.random((m, min(n, 4 * kk))), axis=1)[:, :kk].astype(np.int32)
        a += n - min(n, 4 * kk)
        b += n - min(n, 4 * kk)
        a[m // 2, 0], b[m // 2, -1] = -1, -1
        a[m - 1, 0] = n
        for x, y in zip(lists, (a, b)):
            x.append(y.ravel())
        ref.append(sum(len(np.intersect1d(x, y)) for x, y in zip(a, b)) / (m * kk))
    rec = veda.veda_tile_recall(plan, ks, *(torch.as_tensor(np.concatenate(x)).cuda() for x in lists))
    torch.cuda.synchronize()
    assert np.abs(rec[0].cpu().numpy() - np.asarray(ref)).max() <= 1e-6, (rec, ref)


@pytest.mark.parametrize("dtype,tile_tokens", [("f32", 64), ("bf16", 64), ("bf16", 128)])
def test_tiling_search_errors_and_choice(dtype, tile_tokens):
    # Alg. 1 on synthetic calibration tensors: error table against the oracle, same argmin where the
    # oracle's margin is clear.  Head 0 attends within its own frame only, so the frame-shaped
    # tiling must win it by a wide margin.
    from paper_2605_30325_amd import search
    grid, d, heads, samples = (8, 12, 16), 64, 3, 2
    n = int(np.prod(grid))
    cands = [(4, 4, 4), (1, 8, 8), (16, 2, 2)] if tile_tokens == 64 else [(8, 4, 4), (1, 8, 16), (32, 2, 2)]
    wl = wlm.custom_workload(f"search_{dtype}", heads, d, dtype, grid, False, (25, 100), seed=71, batch=samples)
    dev = torch.device("cuda:0")
    q, k, v = wlm.make_qkv(wl, dev)
    frame = torch.arange(n, device=dev) // (grid[1] * grid[2])
    onehot = torch.zeros((n, d), device=dev)
    onehot[torch.arange(n, device=dev), frame] = 8.0
    q[:, 0] = onehot.to(q.dtype)
    k[:, 0] = onehot.to(k.dtype)
    scale = 1.0 / math.sqrt(d)
    best, table = search.tiling_search(q, k, v, grid, cands, (25, 100), scale, tile_tokens=tile_tokens)
    torch.cuda.synchronize()
    ref = np.zeros_like(table)
    for h in range(heads):
        for b in range(samples):
            ref[h] += vo.tiling_search_errors(hz.to_f32_numpy(q[b, h]), hz.to_f32_numpy(k[b, h]),
                                              hz.to_f32_numpy(v[b, h]), grid, cands, (25, 100), scale)
    _say(f"[parity] tiling search {dtype}: gpu {table.tolist()} oracle {ref.tolist()} best {best.tolist()}")
    # bf16 outputs carry 2^-9 relative rounding on both tensors: an absolute floor per table entry
    floor = samples * n * d * (2.0 ** -8 * 0.5) ** 2 if dtype == "bf16" else 1e-6
    assert np.all(np.abs(table - ref) <= 0.03 * ref + floor), (table, ref)
    assert tuple(best[0]) == cands[1]          # the frame-shaped tiling
    for h in range(heads):
        order = np.sort(ref[h])
        if order[1] - order[0] > 0.1 * order[1] + 2 * floor:
            assert tuple(best[h]) == tuple(cands[int(np.argmin(ref[h]))]), (h, table[h], ref[h])


def test_target_heatmap_at_full_size_sampled_rows():
    # the 32,760-token workload in the configuration bench.py --heatmap times: whole launch on the
    # GPU, oracle on a seeded sample of query tiles (first and last included), all 624 columns
    wl = wlm.WORKLOADS["wan1p3b_480p"]
    dev = torch.device("cuda:0")
    shapes = wlm.tile_shapes(wl)
    q, k, _ = wlm.make_qkv(wl, dev)
    plan = veda.Plan(wl.batch, wl.heads, wl.head_dim, wl.grid, shapes, wl.torch_dtype)
    qt, vm, _ = veda.veda_tile_layout(plan, q, veda.VEDA_TOKEN_MAJOR)
    kt, _, _ = veda.veda_tile_layout(plan, k, veda.VEDA_TOKEN_MAJOR, want_mask=False)
    scale = 1.0 / math.sqrt(wl.head_dim)
    heat = veda.veda_tile_heatmap(plan, qt, kt, vm, scale)
    torch.cuda.synchronize()
    for h in (0, wl.heads - 1):
        shape = tuple(int(x) for x in shapes[h])
        nt, soff = plan.tiles[h], plan.score_offset[h]
        rows = hz.sample_tiles(nt, 6, 100 + h)
        ref = vo.tile_heatmap(hz.to_f32_numpy(q[0, h]), hz.to_f32_numpy(k[0, h]), wl.grid, shape, scale,
                              query_tiles=rows)[rows]
        got = heat[0, soff:soff + nt * nt].view(nt, nt)[torch.as_tensor(rows).to(dev)].cpu().numpy().astype(np.float64)
        rel = np.abs(got - ref) / ref
        _say(f"[parity] {wl.name} head {h}: target scores of {len(rows)} query tiles, max rel err {rel.max():.2e}")
        assert rel.max() <= 2e-4


# ---------------------------------------------------------------- 128-token tiles
@pytest.mark.parametrize("d", [128, 64])
def test_128_token_tiles_whole_path(d):
    # the paper's tile size: every stage against the oracle with 128-token tile shapes whose halves
    # are cut across t, h or w; ragged on every axis; batch 2
    shapes = np.asarray([(8, 4, 4), (2, 8, 8), (32, 2, 2), (1, 8, 16), (1, 1, 128)], np.int32)
    wl = wlm.custom_workload(f"b128_{d}", len(shapes), d, "bf16", (9, 18, 18), True, (25, 100), seed=81, batch=2,
                             latent_dim=32)
    _whole_path_128(wl, shapes)


def _whole_path_128(wl, shapes):
    d = wl.head_dim
    dev = torch.device("cuda:0")
    q, k, v = wlm.make_qkv(wl, dev)
    plan = veda.Plan(wl.batch, wl.heads, d, wl.grid, shapes, wl.torch_dtype, tile_tokens=128)
    eq, ek = wlm.make_estimator(wl, "q"), wlm.make_estimator(wl, "k")
    pq = veda.Mlp(eq.w1, eq.b1, eq.w2, eq.b2, eq.relu, dev)
    pk = veda.Mlp(ek.w1, ek.b1, ek.w2, ek.b2, ek.relu, dev)
    sscale = hz.score_scale_of(wl)
    scale = 1.0 / math.sqrt(d)
    qt, vm, vc = veda.veda_tile_layout(plan, q, veda.VEDA_TOKEN_MAJOR)
    kt, _, _ = veda.veda_tile_layout(plan, k, veda.VEDA_TOKEN_MAJOR, want_mask=False)
    vt, _, _ = veda.veda_tile_layout(plan, v, veda.VEDA_CHANNEL_MAJOR, want_mask=False)
    s, _ = veda.veda_tile_score(plan, qt, kt, vm, pq, pk, sscale)
    kph = np.asarray([max(1, -(-n // 4)) for n in plan.tiles], np.int32)
    rp, ci = veda.veda_tile_select(plan, s, kph)
    out = torch.full((wl.batch, wl.heads, wl.tokens, d), float("nan"), dtype=wl.torch_dtype, device=dev)
    out, lse = veda.veda_sparse_attn_fwd(plan, qt, kt, vt, vm, rp, ci, scale, out=out, want_lse=True)
    torch.cuda.synchronize()
    assert torch.isfinite(out.float()).all()
    # target tile scores over whole 128-token tiles, all rows and then a subset
    heat = veda.veda_tile_heatmap(plan, qt, kt, vm, scale)
    some = np.asarray(sorted({0, plan.total_tiles - 1, plan.tile_offset[wl.heads // 2] + 1}), np.int32)
    part = torch.full_like(heat, -7.0)
    veda.veda_tile_heatmap(plan, qt, kt, vm, scale, torch.as_tensor(some).to(dev), part)
    torch.cuda.synchronize()
    rp_np, ci_np = rp.cpu().numpy(), ci.cpu().numpy()
    vm_np = vm.cpu().numpy().view(np.uint64).reshape(-1, 2)
    queries = np.arange(wl.tokens)
    for b in range(wl.batch):
        for h in range(wl.heads):
            shape = tuple(int(x) for x in shapes[h])
            nt, toff, soff, ksel = plan.tiles[h], plan.tile_offset[h], plan.score_offset[h], int(kph[h])
            assert nt == vo.num_tiles(wl.grid, shape)
            qh, kh, vh = q[b, h], k[b, h], v[b, h]
            ref_q, mask, cnt = vo.tile_layout(hz.raw_numpy(qh), wl.grid, shape)
            assert np.array_equal(hz.raw_numpy(qt[b, toff:toff + nt]).reshape(ref_q.shape), ref_q)
            assert np.array_equal(vm_np[toff:toff + nt], mask)
            assert np.array_equal(vc[toff:toff + nt].cpu().numpy(), cnt)
            ref_v, _, _ = vo.tile_layout(hz.raw_numpy(vh), wl.grid, shape, channel_major=True)   # [nt][d][128]
            got_v = hz.raw_numpy(vt[b, toff:toff + nt]).reshape(nt, 2, d, 64)                     # [nt][2][d][64]
            assert np.array_equal(got_v, ref_v.reshape(nt, d, 2, 64).transpose(0, 2, 1, 3))
            qf, kf, vf = hz.to_f32_numpy(qh), hz.to_f32_numpy(kh), hz.to_f32_numpy(vh)
            lat = []
            for x, e in ((qf, eq), (kf, ek)):
                lat.append(vo.mlp(vo.trippool(x, wl.grid, shape), e.w1[h], e.b1[h], e.w2[h], e.b2[h], e.relu))
            s_ref = vo.score(lat[0], lat[1], np.float32(sscale))
            g_s = s[b, soff:soff + nt * nt].view(nt, nt).cpu().numpy()
            assert np.array_equal(g_s.view(np.uint32), s_ref.view(np.uint32)), (b, h)
            sel = vo.select(s_ref, ksel)
            r0 = b * plan.total_tiles + toff
            lo = int(rp_np[r0])
            assert np.all(np.diff(rp_np[r0:r0 + nt + 1]) == ksel)
            assert np.array_equal(ci_np[lo:lo + nt * ksel].reshape(nt, ksel), sel), (b, h)
            ref, lse_ref, _ = vo.masked_attention(qf, kf, vf, wl.grid, shape, sel, scale, queries, want_stats=True)
            err = np.abs(hz.to_f32_numpy(out[b, h]).astype(np.float64) - ref)
            lerr = np.abs(lse[b, h].cpu().numpy().astype(np.float64) - lse_ref)
            h_ref = vo.tile_heatmap(qf, kf, wl.grid, shape, scale)
            h_got = heat[b, soff:soff + nt * nt].view(nt, nt).cpu().numpy().astype(np.float64)
            rel = (np.abs(h_got - h_ref) / h_ref).max()
            p_got = part[b, soff:soff + nt * nt].view(nt, nt).cpu().numpy()
            listed = np.asarray([g - toff for g in some if toff <= g < toff + nt], np.int64)
            assert np.array_equal(p_got[listed], heat[b, soff:soff + nt * nt].view(nt, nt).cpu().numpy()[listed])
            assert np.all(np.delete(p_got, listed, axis=0) == -7.0)
            _say(f"[parity] {wl.name} b{b} h{h} {shape}: max_abs {err.max():.2e} mean_abs {err.mean():.2e} "
                 f"lse {lerr.max():.2e} heat rel {rel:.2e}")
            assert err.max() <= hz.BF16_MAX_ABS and err.mean() <= hz.BF16_MEAN_ABS and lerr.max() <= 2e-2
            assert rel <= 2e-4


@pytest.mark.parametrize("dtype,d,tile_tokens", [("bf16", 128, 64), ("f32", 64, 64), ("bf16", 64, 128)])
def test_closed_form_scorer_bit_exact(dtype, d, tile_tokens):
    # weight-free scores against the oracle, bit for bit, then their recall against the target scores
    if tile_tokens == 64:
        wl = wlm.custom_workload(f"cf_{dtype}_{d}", 4, d, dtype, (9, 18, 18), True, (25, 100), seed=91)
        shapes = wlm.tile_shapes(wl)
    else:
        shapes = np.asarray([(8, 4, 4), (2, 8, 8), (1, 8, 16), (1, 1, 128)], np.int32)
        wl = wlm.custom_workload(f"cf128_{d}", 4, d, dtype, (9, 18, 18), True, (25, 100), seed=91)
    dev = torch.device("cuda:0")
    q, k, _ = wlm.make_qkv(wl, dev)
    plan = veda.Plan(wl.batch, wl.heads, d, wl.grid, shapes, wl.torch_dtype, tile_tokens=tile_tokens)
    qt, vm, _ = veda.veda_tile_layout(plan, q, veda.VEDA_TOKEN_MAJOR)
    kt, _, _ = veda.veda_tile_layout(plan, k, veda.VEDA_TOKEN_MAJOR, want_mask=False)
    for lam in (0.0, 0.37):
        s, _ = veda.veda_tile_score_closed_form(plan, qt, kt, vm, lam)
        torch.cuda.synchronize()
        for h in range(wl.heads):
            shape = tuple(int(x) for x in shapes[h])
            nt, soff = plan.tiles[h], plan.score_offset[h]
            ref = vo.closed_form_scores(hz.to_f32_numpy(q[0, h]), hz.to_f32_numpy(k[0, h]), wl.grid, shape, lam)
            got = s[0, soff:soff + nt * nt].view(nt, nt).cpu().numpy()
            assert np.array_equal(got.view(np.uint32), ref.view(np.uint32)), (lam, h)
    if tile_tokens == 64:
        kph = wlm.keep_budget(wl, None, shapes)
        heat = veda.veda_tile_heatmap(plan, qt, kt, vm, 1.0 / math.sqrt(d))
        _, ci_t = veda.veda_tile_select(plan, heat, kph)
        _, ci_c = veda.veda_tile_select(plan, s, kph)
        rec = veda.veda_tile_recall(plan, kph, ci_c, ci_t)
        torch.cuda.synchronize()
        _say(f"[parity] {wl.name}: recall of the closed-form scorer against the target scores {rec.cpu().numpy().round(3).tolist()}")
        assert bool((rec > 0.25).all())      # well above the 0.25 keep fraction a blind scorer would get
