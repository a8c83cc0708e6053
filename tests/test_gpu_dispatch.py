"""GPU tests of the size-dependent forms of the kernels, at the sizes where each can go wrong (edges of tiles,
remainders, both sides of a dispatch rule), against the oracle."""
import numpy as np
import pytest

from oracle import ppo_oracle as orc
from paper_2509_16434_amd import configs, synth

from helpers import TOL_BF16, fill_learner, rel_l2

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def L():
    from paper_2509_16434_amd import learner
    return learner


@pytest.mark.parametrize("S", [1, 2, 3, 63, 65, 1023, 1025, 2048, 8191, 8192, 8193])
def test_permutation_one_launch_form(L, S):
    """One block holds up to 8192 units; from 8193 on the bucket kernels take over."""
    np.testing.assert_array_equal(L.permutation_static(S, 77, 3, 2).cpu().numpy(), orc.permutation(77, 3, 2, S))


@pytest.mark.parametrize("hid,N", [(32, 1), (32, 33), (64, 31), (128, 65), (48, 33)])
def test_output_layer_of_act_and_forward(L, hid, N):
    """The fused output layer (widths 32, 64, 128; 32 samples per wave) and the GEMM form (48)."""
    import torch
    cfg = configs.get_config(0, num_envs=N, horizon=1)
    net = cfg["net"]
    net["fc_dim"] = [hid]
    ro = synth.rollout(cfg)
    params = synth.init_params(net, 5)
    a0, a1, _ = synth.param_slices(net)["logstd"]
    params[a0:a1] = np.linspace(-0.5, 0.5, net["act_dim"], dtype=np.float32)
    lrn = L.Learner(net, N, 1, "fp32")
    lrn.set_params(params)
    noise = np.random.default_rng(1).standard_normal((N, net["act_dim"])).astype(np.float32)
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    a, lp, v = (x.cpu().numpy() for x in lrn.act(0, dev(ro["obs"][0]), dev(ro["proprio"][0]), dev(noise)))
    oa, olp, ov = orc.act(net, params, ro["obs"][0], ro["proprio"][0], noise)
    omu = oa - np.exp(params[a0:a1].astype(np.float64)) * noise
    assert np.linalg.norm(a - oa) / np.linalg.norm(omu) <= TOL_BF16 and rel_l2(v, ov) <= TOL_BF16 and np.max(np.abs(lp - olp)) <= 1e-3
    fill_learner(lrn, cfg, ro)
    mu, v2 = (x.cpu().numpy() for x in lrn.forward())
    assert rel_l2(mu, omu) <= TOL_BF16 and rel_l2(v2, ov) <= TOL_BF16


@pytest.mark.parametrize("M,N,K", [(1, 3, 8), (33, 40, 136), (512, 1024, 512), (65, 32, 2048), (64, 64, 1056),   # 32 x 32 tiles
                                   (1250, 256, 4480), (129, 72, 4168), (4100, 32, 2056), (700, 40, 3000),       # slices of K
                                   (4096, 512, 10304), (8400, 130, 4104), (256, 4096, 2048)])
def test_gemm_plans(L, M, N, K):
    """Products with plain rows in each form plan_gemm can choose: ragged rows, columns and last slices."""
    rng = np.random.default_rng(M + N + K)
    a = synth.narrow_bf16(rng.standard_normal((M, K), dtype=np.float32))
    b = synth.narrow_bf16(rng.standard_normal((N, K), dtype=np.float32))
    want = a @ b.T
    assert np.abs(L.diag_gemm(a, b) - want).max() <= 1e-4 * np.abs(want).max()


def _check_gradients(L, cfg, N, T, change=None):
    """One minibatch of a conditioned rollout: every tensor's gradient against the oracle's bf16-operand mode (`change`:
    edits the initial parameters in place)."""
    import torch
    net, hp = cfg["net"], dict(cfg["hp"], epochs=1, minibatches=1, seed=3)
    ro = synth.rollout(cfg, conditioned=True)
    params = synth.init_params(net, 9)
    if change:
        change(params)
    lrn = L.Learner(net, N, T, cfg["obs_dtype"])
    lrn.set_params(params)
    distill = cfg["kind"] == "distill"
    fill_learner(lrn, cfg, ro, distill=distill)
    fr = {k: v.reshape((N * T,) + v.shape[2:]) for k, v in ro.items() if k != "last_value"}
    if distill:
        lrn.distill_update(hp)
        with orc.quant(1):
            _, qg = orc.distill_loss_grad(net, params, fr["obs"], fr["proprio"], fr["action"])
    else:
        lrn.gae(torch.from_numpy(ro["last_value"]).cuda(), hp["gamma"], hp["lam"])
        adv, ret = (x.cpu().numpy().reshape(-1) for x in lrn.get_adv_ret())
        lrn.update(hp)
        with orc.quant(1):
            _, qg = orc.ppo_loss_grad(net, params, fr["obs"], fr["proprio"], fr["action"], fr["logp_old"], fr["value"], adv, ret,
                                      clip_eps=hp["clip_eps"], vclip_eps=hp["vclip_eps"], vf_coef=hp["vf_coef"], ent_coef=hp["ent_coef"])
    g = lrn.get_grads()
    bad = {n: rel_l2(g[a:b], qg[a:b]) for n, (a, b, _) in synth.param_slices(net).items() if rel_l2(g[a:b], qg[a:b]) > TOL_BF16}
    assert not bad, bad


def _check_forward(L, cfg, N, T):
    """Action means and values of some stored samples, chosen by index, against the oracle."""
    import torch
    net, ro = cfg["net"], synth.rollout(cfg, conditioned=True)
    params = synth.init_params(net, 9)
    lrn = L.Learner(net, N, T, cfg["obs_dtype"])
    lrn.set_params(params)
    fill_learner(lrn, cfg, ro)
    idx = np.random.default_rng(1).permutation(N * T)[: max(1, N * T // 2)].astype(np.int32)
    mu, v = (x.cpu().numpy() for x in lrn.forward(torch.from_numpy(idx).cuda()))
    with orc.quant(1):
        omu, ov = orc.forward(net, params, ro["obs"].reshape((N * T,) + ro["obs"].shape[2:])[idx], ro["proprio"].reshape(N * T, -1)[idx])
    assert rel_l2(mu, omu) <= TOL_BF16 and rel_l2(v, ov) <= TOL_BF16


@pytest.mark.parametrize("hid,A,N,T,kind", [(64, 1, 9, 7, "ppo"), (32, 7, 8, 8, "ppo"), (128, 8, 5, 13, "ppo"), (64, 9, 16, 16, "ppo"), (128, 23, 31, 5, "ppo"),
                                            (64, 31, 11, 6, "ppo"), (64, 1, 9, 7, "distill"), (128, 16, 5, 13, "distill"), (32, 25, 3, 43, "distill")])
def test_output_layer_and_loss(L, hid, A, N, T, kind):
    """Output layer, loss and their backward in one kernel: eight columns per lane, 64 samples per block, with remainders of both."""
    cfg = configs.get_config(0, num_envs=N, horizon=T)
    cfg["net"].update(fc_dim=[hid], act_dim=A)
    if kind == "distill":
        cfg["kind"], cfg["net"]["has_value_head"] = "distill", 0
    _check_gradients(L, cfg, N, T)


@pytest.mark.parametrize("kind,A,hp", [("ppo", 7, {}), ("ppo", 23, dict(vclip_eps=0.05, clip_eps=0.05, ent_coef=0.01)), ("distill", 9, {}), ("distill", 23, dict(aux_dim=3, aux_coef=0.5))])
def test_both_kernels_of_the_loss_agree(L, kind, A, hp):
    """72 hidden units of which eight have no weights compute what 64 do, but their loss is taken one lane per sample behind a product of
    its own, not four lanes per sample beside it: statistics and gradients of one batch through both.  Both take the same bf16
    operands; their fp32 sums differ in order (a few 1e-6), and a gradient's bf16 rounding may go the other way (2^-8 of one value
    in some thousand, hence 1e-3 of a tensor)."""
    import torch
    N, T, got = 70, 3, {}
    for hid in (64, 72):
        cfg = configs.get_config(1, num_envs=N, horizon=T)
        net = cfg["net"]
        net.update(in_h=24, in_w=32, fc_dim=[hid], act_dim=A, has_value_head=int(kind == "ppo"))
        cfg["kind"] = kind
        sl = synth.param_slices(net)
        narrow = dict(net, fc_dim=[64])
        p64 = synth.init_params(narrow, 9)
        params = np.zeros(max(b for _, b, _ in sl.values()), np.float32)
        live = {}
        for n, (a, b, shape) in synth.param_slices(narrow).items():
            at = np.arange(sl[n][0], sl[n][1]).reshape(sl[n][2])[tuple(slice(0, k) for k in shape)]
            live[n] = at
            params[at.reshape(-1)] = p64[a:b]
        ro = synth.rollout(dict(cfg, net=narrow), conditioned=True)
        lrn = L.Learner(net, N, T, cfg["obs_dtype"])
        lrn.set_params(params)
        fill_learner(lrn, cfg, ro, distill=kind == "distill")
        h = dict(cfg["hp"], epochs=1, minibatches=1, seed=3, **hp)
        if kind == "ppo":
            lrn.gae(torch.from_numpy(ro["last_value"]).cuda(), h["gamma"], h["lam"])
        st = (lrn.update if kind == "ppo" else lrn.distill_update)(h)[0]
        g = lrn.get_grads()
        got[hid] = (np.array([st[f] for f in L.STAT_FIELDS]), {n: g[at.reshape(-1)] for n, at in live.items()})
    np.testing.assert_allclose(got[64][0], got[72][0], rtol=2e-5, atol=2e-6)
    bad = {n: rel_l2(got[64][1][n], x) for n, x in got[72][1].items() if rel_l2(got[64][1][n], x) > 1e-3}
    assert not bad, bad


@pytest.mark.parametrize("ci,h,w", [(1, 51, 61), (1, 49, 58), (1, 89, 117), (1, 31, 33), (1, 45, 90), (3, 49, 58), (2, 62, 101)])
def test_gradients_odd_second_layer_width(L, ci, h, w):
    """Widths whose first-layer output is odd."""
    cfg = configs.get_config(ci, num_envs=12, horizon=4)
    cfg["net"].update(in_h=h, in_w=w)
    _check_gradients(L, cfg, 12, 4)


@pytest.mark.parametrize("ci,h,w", [(1, 20, 193), (1, 18, 261), (1, 37, 390), (2, 34, 322), (2, 64, 410), (2, 33, 262)])
def test_gradients_wide_rows(L, ci, h, w):
    """Rows too long for a row-wise LDS image (more than 48 pixels of 64 channels): tiles of columns, with a last column tile that
    is full, ragged or ends in an odd pixel; 64 x 128 tiles of the last layer from 52-pixel rows.  (The second layer, of 32
    channels, makes its rows from the images here.)"""
    cfg = configs.get_config(ci, num_envs=6, horizon=4)
    cfg["net"].update(in_h=h, in_w=w)
    _check_gradients(L, cfg, 6, 4)


@pytest.mark.parametrize("conv,more,h,w", [((16, 32, 64, 32), {}, 18, 404), ((32, 128, 64), {}, 20, 200), ((32, 64, 64), dict(embed_dim=32), 18, 261),
                                           ((16, 32, 32, 16), {}, 33, 437)])
def test_gradients_wide_rows_of_a_stored_layer(L, conv, more, h, w):
    """Rows of more than 96 pixels of 32 channels that come from memory, with the sign bits of their results: a deeper layer, a second
    layer of more than 64 channels, a network with an embedding."""
    cfg = configs.get_config(1, num_envs=6, horizon=4)
    cfg["net"].update(dict(in_h=h, in_w=w, conv_ch=list(conv)), **more)
    _check_gradients(L, cfg, 6, 4)


@pytest.mark.parametrize("ci,conv,more,h,w,N,T", [
    (1, (32, 64, 64), {}, 52, 76, 20, 7),                              # 7 x 10 results: bands of up to six rows over the images' borders
    (1, (32, 64, 64), {}, 28, 28, 150, 2), (1, (32, 64, 64), {}, 32, 29, 60, 5),  # 4 x 4: several images per band (of even and odd heights)
    (1, (32, 64, 64, 64), {}, 36, 44, 75, 4),                          # odd heights 9 and 5
    (1, (32, 64, 64, 128), {}, 60, 50, 100, 3),                        # to 128 channels
    (3, (32, 64, 64, 128), {}, 52, 40, 50, 3), (3, (32, 64, 64, 64), {}, 64, 44, 30, 5),   # two views: strided features
    (1, (32, 64, 64), dict(embed_dim=32), 44, 52, 45, 4),              # dense features
    (1, (16, 32, 64), dict(layer_norm=1), 28, 28, 150, 2), (1, (16, 32, 64, 64), dict(layer_norm=1), 32, 36, 75, 4)])  # unmasked, 32 channels from memory
def test_stacked_bands(L, ci, conv, more, h, w, N, T):
    """Bands of rows that run on over the images' borders: even and odd heights, a band of several images, strided features."""
    cfg = configs.get_config(ci, num_envs=N, horizon=T)
    cfg["net"].update(dict(in_h=h, in_w=w, conv_ch=list(conv)), **more)
    _check_gradients(L, cfg, N, T)


@pytest.mark.parametrize("ci,conv,h,w,N,T", [
    (1, (32, 64, 64), 28, 28, 1500, 4), (1, (32, 64, 64, 64), 36, 44, 600, 4),   # 4 x 4; odd heights 9 and 5
    (1, (32, 64, 64, 128), 60, 50, 1200, 2), (3, (32, 64, 64, 128), 28, 36, 1100, 2)])   # to 128 channels; two views
def test_stacked_bands_many_per_block(L, ci, conv, h, w, N, T):
    """The same with several tiles for each block, more than its ring has buffers in the narrow layers."""
    cfg = configs.get_config(ci, num_envs=N, horizon=T)
    cfg["net"].update(in_h=h, in_w=w, conv_ch=list(conv), fc_dim=[32])
    _check_gradients(L, cfg, N, T)


@pytest.mark.parametrize("c0,views,conv,h,w", [(1, 1, (32, 64), 9, 10), (1, 1, (32, 64, 16), 16, 8), (1, 1, (32, 64, 64), 21, 67),
                                               (1, 2, (32, 64, 64), 45, 90), (1, 1, (32, 64, 64), 13, 333), (1, 1, (32, 64, 64), 35, 280),
                                               (3, 1, (32, 64), 11, 14), (3, 2, (32, 64, 32), 30, 71), (3, 1, (32, 64, 64), 14, 200)])
def test_first_two_convolutions_in_one_kernel(L, c0, views, conv, h, w):
    """The second layer's kernels that make the first layer's output in LDS: tiles of few and of many pixel groups, one and several
    bands, tiles of columns, a last band or column that ends inside a tile, the result in the feature matrix (two layers)."""
    cfg = configs.get_config(1, num_envs=10, horizon=4)
    cfg["net"].update(in_c=c0, n_views=views, in_h=h, in_w=w, conv_ch=list(conv))
    _check_gradients(L, cfg, 10, 4)


@pytest.mark.parametrize("c0,views,conv,h,w,N", [(1, 1, (32, 64, 64), 28, 31, 425), (1, 1, (32, 64), 21, 67, 410), (1, 1, (32, 64, 64), 13, 333, 130),
                                                 (1, 1, (32, 64), 45, 90, 150), (1, 1, (32, 64, 32), 12, 34, 450), (3, 2, (32, 64, 32), 30, 71, 100),
                                                 (3, 1, (32, 64), 30, 270, 90), (3, 1, (32, 64, 64), 52, 100, 130)])
def test_first_two_convolutions_over_many_tiles(L, c0, views, conv, h, w, N):
    """The same kernels with six to nine tiles per block (a tile is a whole small image, one of two to four bands, one of three or five
    columns): the rings of images and gradients and the two row buffers turn over, mask stores lie between the loads that are
    waited for, the weight gradient deals its loads between the groups.  All producing waves with three groups or fewer (28x31,
    12x34, RGB 30x71), or four and five; odd widths, rounded-up mask rows (12x34, 45x90)."""
    cfg = configs.get_config(1, num_envs=N, horizon=4)
    cfg["net"].update(in_c=c0, n_views=views, in_h=h, in_w=w, conv_ch=list(conv), fc_dim=[64])
    _check_gradients(L, cfg, N, 4)


@pytest.mark.parametrize("conv,ln,h,w", [((32, 16), 0, 24, 33), ((32, 32, 64), 1, 40, 66), ((32, 128), 0, 29, 80), ((32, 128, 64), 1, 35, 42)])
def test_weight_gradient_dealt_by_halves(L, conv, ln, h, w):
    """32 input channels: the last k-tile and the bias column go to the waves by halves of 64 output channels; fewer than 32 of them,
    one half, two blocks of 64, behind made rows and behind stored ones (layer normalisation)."""
    cfg = configs.get_config(1, num_envs=10, horizon=4)
    cfg["net"].update(in_h=h, in_w=w, conv_ch=list(conv), layer_norm=ln)
    _check_gradients(L, cfg, 10, 4)


@pytest.mark.parametrize("ci,h,w", [(1, 12, 34), (1, 27, 50), (1, 40, 61), (1, 21, 147), (3, 20, 35), (3, 33, 106)])
def test_input_gradient_of_a_rounded_up_width(L, ci, h, w):
    """First-layer outputs whose width is no multiple of 8: 17, 25, 31, 74; 18 and 53 (RGB)."""
    cfg = configs.get_config(ci, num_envs=10, horizon=4)
    cfg["net"].update(in_h=h, in_w=w)
    _check_gradients(L, cfg, 10, 4)


@pytest.mark.parametrize("h,w", [(13, 152), (13, 154), (20, 156), (20, 157), (13, 159), (30, 160), (13, 162)])
def test_input_gradient_beside_the_width_known_at_compile_time(L, h, w):
    """First-layer outputs of 76 to 81 columns: 77 to 80 are stored 80 wide, with 39 or 40 columns of the gradient behind them, of
    which the form with the width known at compile time takes 40."""
    cfg = configs.get_config(1, num_envs=10, horizon=4)
    cfg["net"].update(in_h=h, in_w=w)
    _check_gradients(L, cfg, 10, 4)


@pytest.mark.parametrize("c0,h,w,N", [(1, 37, 50, 700), (3, 37, 50, 700), (1, 60, 97, 500), (3, 52, 100, 480), (1, 24, 390, 260), (3, 30, 270, 300)])
def test_non_finite_pixels_stay_in_their_sample(L, c0, h, w, N):
    """Values beside a window are read with it, LDS keeps those of earlier tiles, and neither must reach a sum: NaN and infinity in
    some samples' images leave every other sample's outputs as they were, bit for bit.  A block makes five tiles or more, of
    good and bad samples in turn; whole rows in two and in three bands, and tiles of columns."""
    import torch
    cfg = configs.get_config(1, num_envs=N, horizon=1)
    cfg["net"].update(in_c=c0, in_h=h, in_w=w)
    ro = synth.rollout(cfg)
    rng = np.random.default_rng(5)
    bad = np.flatnonzero(rng.random(N) < 0.3)
    outs = []
    for spoil in (False, True):
        if spoil:
            for i in bad:
                ro["obs"][0, i, 0, :, rng.integers(h), rng.integers(w)] = np.nan
                ro["obs"][0, i, 0, :, rng.integers(h), 0] = np.inf
                ro["obs"][0, i, 0, :, :, w - 1] = -np.inf
        lrn = L.Learner(cfg["net"], N, 1, "fp32")
        lrn.set_params(synth.init_params(cfg["net"], 4))
        fill_learner(lrn, dict(cfg, obs_dtype="fp32"), ro)
        outs.append([x.cpu().numpy() for x in lrn.forward()])
    keep = np.setdiff1d(np.arange(N), bad)
    assert len(bad) > N // 5
    for a, b in zip(*outs):
        np.testing.assert_array_equal(a[keep], b[keep])
        assert np.isfinite(a).all() and (a[bad] != b[bad]).any()


@pytest.mark.parametrize("c0,conv,h,w,N", [(1, (32, 64, 64), 37, 50, 100), (1, (32, 64, 64), 12, 34, 100), (1, (32, 64, 64, 128), 60, 97, 40), (1, (32, 64, 64), 24, 390, 40),
                                           (3, (32, 64, 64), 37, 50, 100), (3, (32, 64, 32), 30, 270, 40), (1, (32, 64, 64), 20, 157, 60)])
def test_gradients_after_a_non_finite_update(L, c0, conv, h, w, N):
    """An update of another learner whose images are all NaN leaves NaN in LDS and in the memory it gives back; the gradients of the
    next learner are those of before, bit for bit (slots, pads and slack that a kernel reads are ones that it has written)."""
    import torch
    cfg = configs.get_config(1, num_envs=N, horizon=2)
    net, hp = cfg["net"], dict(cfg["hp"], epochs=1, minibatches=1, seed=3)
    net.update(in_c=c0, in_h=h, in_w=w, conv_ch=list(conv), fc_dim=[64])
    ro = synth.rollout(cfg, conditioned=True)
    params = synth.init_params(net, 9)

    def gradients(rollout):
        lrn = L.Learner(net, N, 2, cfg["obs_dtype"])
        lrn.set_params(params)
        fill_learner(lrn, cfg, rollout)
        lrn.gae(torch.from_numpy(rollout["last_value"]).cuda(), hp["gamma"], hp["lam"])
        lrn.update(hp)
        return lrn.get_grads()

    before = gradients(ro)
    assert not np.array_equal(before, gradients(dict(ro, obs=np.full_like(ro["obs"], np.nan))), equal_nan=True)
    np.testing.assert_array_equal(before, gradients(ro))


@pytest.mark.parametrize("conv,h,w,N,more", [((16, 32, 64), 40, 48, 300, dict(layer_norm=1)), ((16, 32, 64), 84, 90, 260, dict(layer_norm=1)), ((16, 32), 118, 157, 130, dict(layer_norm=1)),
                                             ((16, 32), 20, 28, 700, {}), ((16, 32, 64), 37, 53, 300, {}), ((32, 64, 64), 28, 28, 900, {}), ((32, 64, 64, 64), 36, 44, 600, {}),
                                             ((8, 16), 32, 32, 600, dict(fc_dim=[64])), ((8, 16), 28, 33, 1000, dict(fc_dim=[32]))])
def test_non_finite_images_in_the_fused_and_stacked_kernels(L, conv, h, w, N, more):
    """First layer with its normalisation, 16 -> 32 channels, bands over the images' borders, the small network in one kernel: images
    that are NaN or hold infinities leave the other samples' outputs as they were, bit for bit, by index and in the policy step,
    and a learner whose images are all NaN leaves the next learner's gradients as they were."""
    import torch
    cfg = configs.get_config(1, num_envs=N, horizon=1)
    net, hp = cfg["net"], dict(cfg["hp"], epochs=1, minibatches=1, seed=3)
    net.update(dict(in_h=h, in_w=w, conv_ch=list(conv)), **more)
    ro = synth.rollout(cfg, conditioned=True)
    params = synth.init_params(net, 4)
    bad = np.arange(1, N, 3)
    spoiled = ro["obs"].copy()
    spoiled[0, bad] = np.nan
    spoiled[0, bad[::2], ..., : h // 2, :] = 1.0
    spoiled[0, bad[::3], ..., h - 1, w // 2] = -np.inf
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    noise = torch.zeros(N, net["act_dim"], device="cuda")

    def run(obs):
        lrn = L.Learner(net, N, 1, "fp32")
        lrn.set_params(params)
        fill_learner(lrn, dict(cfg, obs_dtype="fp32"), dict(ro, obs=obs))
        outs = list(lrn.forward(torch.arange(N, device="cuda", dtype=torch.int32)))
        lrn.gae(dev(ro["last_value"]), hp["gamma"], hp["lam"])
        lrn.update(hp)
        g = lrn.get_grads()
        lrn.set_params(params)
        return [x.cpu().numpy() for x in outs + list(lrn.act(0, dev(obs[0]), dev(ro["proprio"][0]), noise))], g

    outs, g = run(ro["obs"])
    sick, _ = run(spoiled)
    run(np.full_like(spoiled, np.nan))
    again, g2 = run(ro["obs"])
    keep = np.setdiff1d(np.arange(N), bad)
    for a, b, c in zip(outs, sick, again):
        np.testing.assert_array_equal(a[keep], b[keep])
        np.testing.assert_array_equal(a, c)
    np.testing.assert_array_equal(g, g2)


@pytest.mark.parametrize("c0,conv,h,w", [(1, (32, 64, 32), 22, 226), (1, (8, 16), 33, 47), (1, (16, 32, 64, 128), 40, 64), (1, (32, 64), 16, 130), (1, (64, 64), 21, 24),
                                         (3, (16, 32), 18, 66), (3, (32, 64, 64), 37, 53), (1, (16, 64), 9, 16)])
def test_gradients_with_layer_norm(L, c0, conv, h, w):
    """Convolutions that store their output before a layer normalisation: the first layer's weight gradient from a stored
    gradient (rows of one ragged 32-pixel step, several steps, several bands), unmasked transposed convolutions."""
    cfg = configs.get_config(1, num_envs=10, horizon=4)
    cfg["net"].update(in_c=c0, in_h=h, in_w=w, conv_ch=list(conv), layer_norm=1)
    _check_gradients(L, cfg, 10, 4)


@pytest.mark.parametrize("ci,conv,h,w,N,T", [(1, (16, 32), 16, 16, 3, 1), (1, (16, 16), 20, 24, 100, 3), (1, (16, 32), 33, 30, 7, 2), (1, (16, 32, 32), 41, 69, 90, 3),
                                              (1, (16, 32), 64, 80, 5, 3), (1, (16, 32, 64), 84, 90, 4, 2), (1, (16, 32, 64), 120, 160, 3, 2),
                                              (1, (16, 32, 64), 122, 160, 3, 2), (1, (16, 32), 2, 64, 5, 3)])
def test_first_layer_and_its_normalisation(L, ci, conv, h, w, N, T):
    """First convolution, normalisation and ReLU in one kernel per direction: ten, twenty or 38 tiles per wave at most, rows that are no
    multiple of four pixels, several images per block (with ten; the others in the next test), and one row more than the registers
    hold (the separate kernels)."""
    cfg = configs.get_config(ci, num_envs=N, horizon=T)
    cfg["net"].update(in_h=h, in_w=w, conv_ch=list(conv), layer_norm=1)
    _check_gradients(L, cfg, N, T)


@pytest.mark.parametrize("views,conv,h,w,N,T", [(1, (16, 32), 84, 90, 257, 2), (1, (16, 32), 84, 96, 300, 2), (2, (16, 32), 83, 91, 130, 2),
                                                (1, (16, 32), 118, 157, 131, 2), (1, (16, 32), 120, 160, 131, 2), (2, (16, 32), 119, 150, 65, 2),
                                                (2, (16, 32), 41, 69, 129, 2)])
def test_several_images_per_block_of_the_first_layer_and_its_normalisation(L, views, conv, h, w, N, T):
    """Blocks with two images or three in the forms with twenty and 38 tiles per wave, rows that are multiples of four pixels and
    others, one view and two: the image and the gradient that travel while the one before is worked on, and sums over images."""
    cfg = configs.get_config(1, num_envs=N, horizon=T)
    cfg["net"].update(in_h=h, in_w=w, conv_ch=list(conv), layer_norm=1, n_views=views, fc_dim=[32])
    _check_gradients(L, cfg, N, T)


@pytest.mark.parametrize("P", [4096, 4104, 8200])
@pytest.mark.parametrize("views,more", [(1, {}), (2, {}), (2, dict(embed_dim=16))])
def test_wide_proprioception_behind_the_first_layer_and_its_normalisation(L, views, more, P):
    """That kernel copies the proprioception too: as many 16-byte pieces as a block has threads, one more, and some twice as many,
    in the forward of the update and in that by index."""
    cfg = configs.get_config(1, num_envs=9, horizon=3)
    cfg["net"].update(dict(in_h=16, in_w=24, conv_ch=[16, 32], layer_norm=1, n_views=views, proprio_dim=P, fc_dim=[32]), **more)
    _check_gradients(L, cfg, 9, 3)
    _check_forward(L, cfg, 9, 3)


@pytest.mark.parametrize("conv,ln,h,w,N,T", [((16, 32, 64, 128), 1, 60, 80, 16, 4), ((16, 32, 32), 1, 37, 53, 20, 7), ((16, 16, 32), 1, 30, 62, 5, 3), ((16, 8, 32), 1, 40, 34, 5, 2),
                                              ((16, 32, 64), 0, 44, 60, 6, 3), ((16, 32), 1, 18, 380, 3, 2), ((16, 32), 1, 18, 390, 3, 2), ((16, 32, 32), 1, 12, 20, 40, 8)])
def test_second_layer_of_sixteen_channels(L, conv, ln, h, w, N, T):
    """16 -> 32 channels from memory: odd heights and widths, last bands of fewer rows, rows up to and beyond the kernels' longest, fewer
    than 32 channels (input gradient: the implicit form), bands of fewer than four rows (forward: the same)."""
    cfg = configs.get_config(1, num_envs=N, horizon=T)
    cfg["net"].update(in_h=h, in_w=w, conv_ch=list(conv), layer_norm=ln)
    _check_gradients(L, cfg, N, T)


@pytest.mark.parametrize("ln", [0, 1])
@pytest.mark.parametrize("h,w,N,T", [(20, 28, 650, 4), (40, 160, 300, 2), (29, 71, 350, 4)])
def test_second_layer_of_sixteen_channels_many_tiles_per_block(L, ln, h, w, N, T):
    """The same with more tiles for a block than its ring has buffers: one, two and four bands per image."""
    cfg = configs.get_config(1, num_envs=N, horizon=T)
    cfg["net"].update(in_h=h, in_w=w, conv_ch=[16, 32], layer_norm=ln, fc_dim=[32])
    _check_gradients(L, cfg, N, T)


@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf])
@pytest.mark.parametrize("conv,h,w,views,more", [((16, 32), 40, 48, 1, {}), ((16, 32), 40, 50, 2, dict(embed_dim=32)), ((16, 32, 64), 118, 157, 1, {}),  # fused
                                                 ((32, 64), 40, 48, 1, {}), ((16, 32), 122, 160, 1, {})])                             # kernels of their own
def test_non_finite_images_before_a_normalisation(L, conv, h, w, views, more, value):
    """One such pixel makes the normalised layer of its image zero, in both forms of that layer: the outputs of every sample are
    the oracle's, and so are the gradients of the layers behind it."""
    import torch
    N = 12
    cfg = configs.get_config(1, num_envs=N, horizon=1)
    net = cfg["net"]
    net.update(dict(in_h=h, in_w=w, conv_ch=list(conv), layer_norm=1, n_views=views, fc_dim=[64]), **more)
    hp = dict(cfg["hp"], epochs=1, minibatches=1, seed=3)
    ro = synth.rollout(cfg, conditioned=True)
    ro["obs"][0, 1::4, -1, 0, h // 2, w // 3] = value
    params = synth.init_params(net, 9)
    lrn = L.Learner(net, N, 1, cfg["obs_dtype"])
    lrn.set_params(params)
    fill_learner(lrn, cfg, ro)
    mu, v = (x.cpu().numpy() for x in lrn.forward())
    lrn.gae(torch.from_numpy(ro["last_value"]).cuda(), hp["gamma"], hp["lam"])
    adv, ret = (x.cpu().numpy().reshape(-1) for x in lrn.get_adv_ret())
    lrn.update(hp)
    g = lrn.get_grads()
    with orc.quant(1):
        omu, ov = orc.forward(net, params, ro["obs"][0], ro["proprio"][0])
        _, qg = orc.ppo_loss_grad(net, params, *(ro[k][0] for k in ("obs", "proprio", "action", "logp_old", "value")), adv, ret,
                                  clip_eps=hp["clip_eps"], vclip_eps=hp["vclip_eps"], vf_coef=hp["vf_coef"], ent_coef=hp["ent_coef"])
    assert rel_l2(mu, omu) <= TOL_BF16 and rel_l2(v, ov) <= TOL_BF16
    behind = {n: rel_l2(g[a:b], qg[a:b]) for n, (a, b, _) in synth.param_slices(net).items() if not n.startswith(("conv0", "ln0"))}
    assert all(e <= TOL_BF16 for e in behind.values()), behind


@pytest.mark.parametrize("chunks", range(1, 21))
def test_layer_norm_backward_of_any_chunk_count(L, chunks):
    """One form of the layer-normalisation backward per number of 16-byte chunks a thread holds (up to 19; 20 reads
    twice): the first layer's 16 x (16 chunks - 0 .. 2) x 16 values fill the last chunk or part of it."""
    cfg = configs.get_config(1, num_envs=10, horizon=2)
    cfg["net"].update(in_h=32, in_w=32 * chunks - 2 * (chunks % 3), conv_ch=[16, 8], fc_dim=[32], layer_norm=1)
    _check_gradients(L, cfg, 10, 2)


@pytest.mark.parametrize("ci,dtype", [(0, "fp32"), (0, "bf16"), (3, "fp32"), (3, "bf16")])
@pytest.mark.parametrize("h,w", [(5, 7), (6, 8), (4, 9), (3, 15), (9, 33)])
def test_stored_images_bit_exact_at_any_width(L, ci, dtype, h, w):
    """Stored rows are padded to multiples of 8 pixels: whole groups, a ragged last group, rows at odd addresses."""
    import torch
    cfg = configs.get_config(ci, num_envs=13, horizon=2)
    cfg["net"].update(in_h=h, in_w=w)
    net = cfg["net"]
    lrn = L.Learner(net, 13, 2, dtype)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(w)
    for t in (1, 0):
        obs = torch.randn(13, net["n_views"], net["in_c"], h, w, generator=gen, device="cuda").to(torch.float32 if dtype == "fp32" else torch.bfloat16)
        z = torch.zeros(13, device="cuda")
        lrn.buffer_write(t, obs, torch.zeros(13, net["proprio_dim"], device="cuda"), torch.zeros(13, net["act_dim"], device="cuda"), z, z, z, z.to(torch.uint8))
        assert torch.equal(lrn.buffer_read_obs(t), obs.to(torch.bfloat16))


@pytest.mark.parametrize("ci", [0, 3])
@pytest.mark.parametrize("h,w,off,cnt", [(5, 7, 3, 1), (4, 9, 1, 11), (6, 8, 5, 2), (9, 33, 0, 12), (16, 16, 4, 8)])
def test_a_range_of_environments_leaves_the_others(L, ci, h, w, off, cnt):
    """Images of a range end inside a wave's staged pieces: nothing before or behind them changes, in the step or the next."""
    import torch
    cfg = configs.get_config(ci, num_envs=13, horizon=2)
    cfg["net"].update(in_h=h, in_w=w)
    net = cfg["net"]
    lrn = L.Learner(net, 13, 2, "bf16")
    gen = torch.Generator(device="cuda")
    gen.manual_seed(w + cnt)
    obs = torch.randn(2, 13, net["n_views"], net["in_c"], h, w, generator=gen, device="cuda").to(torch.bfloat16)
    for t in (0, 1):
        for lo, hi in ((0, off), (off + cnt, 13), (off, off + cnt)):  # the range last, between environments that are there
            z = torch.zeros(hi - lo, device="cuda")
            if hi > lo:
                lrn.buffer_write_range(t, lo, obs[t, lo:hi].contiguous(), torch.zeros(hi - lo, net["proprio_dim"], device="cuda"),
                                       torch.zeros(hi - lo, net["act_dim"], device="cuda"), z, z, z, z.to(torch.uint8))
    assert torch.equal(lrn.buffer_read_obs(0), obs[0]) and torch.equal(lrn.buffer_read_obs(1), obs[1])


@pytest.mark.parametrize("fc,P,N,T", [([96, 40], 8, 50, 4), ([200, 72], 40, 33, 3), ([520, 136, 24], 16, 70, 3), ([264, 512], 8, 31, 1), ([512, 520], 24, 40, 4)])
def test_hidden_layers_weight_and_input_gradient_together(L, fc, P, N, T):
    """Blocks of 128, 256 and 384 columns of the weight gradient beside 32 x 32 tiles of the input gradient: ragged rows, columns
    and depths, one row tile, the deepest (512 outputs) and the first depth that takes two launches (520)."""
    cfg = configs.get_config(1, num_envs=N, horizon=T)
    cfg["net"].update(in_h=32, in_w=32, fc_dim=fc, proprio_dim=P)
    _check_gradients(L, cfg, N, T)


@pytest.mark.parametrize("layers,units,N,T,P", [(2, 64, 33, 5, 8), (1, 96, 70, 3, 40), (3, 32, 9, 4, 16), (2, 24, 40, 4, 8), (4, 32, 130, 2, 8), (2, 160, 65, 1, 8), (2, 64, 200, 6, 8)])
def test_gradients_recurrent(L, layers, units, N, T, P):
    """LSTM layers side by side (units in multiples of 32; up to 64 environments: 64 x 64 tiles, more: 128 x 128) and one
    after the other (24 units): one minibatch with episode ends and initial states against the oracle's
    bf16-operand mode (a wide clip range: no sample sits on a decision)."""
    import torch
    cfg = configs.get_config(1, num_envs=N, horizon=T)
    cfg["net"].update(in_h=16, in_w=20, conv_ch=[8, 16], fc_dim=[32], proprio_dim=P, embed_dim=16, layer_norm=1, lstm_layers=layers, lstm_units=units)
    net, hp = cfg["net"], dict(cfg["hp"], epochs=1, minibatches=1, seed=3, clip_eps=1e3)
    ro = synth.rollout(cfg, conditioned=True)
    rng = np.random.default_rng(units)
    ro["done"] = (rng.random((T, N)) < 0.1).astype(np.uint8)
    h0, c0 = (0.3 * rng.standard_normal((2, layers, N, units))).astype(np.float32)
    params = synth.init_params(net, 4)
    lrn = L.Learner(net, N, T, "bf16")
    lrn.set_params(params)
    fill_learner(lrn, cfg, ro)
    lrn.buffer_write_state(torch.from_numpy(h0).cuda(), torch.from_numpy(c0).cuda())
    lrn.gae(torch.from_numpy(ro["last_value"]).cuda(), hp["gamma"], hp["lam"])
    lrn.update(hp)
    adv, ret = orc.gae(ro["reward"], ro["done"], ro["value"], ro["last_value"], hp["gamma"], hp["lam"])
    with orc.quant(1):
        _, qg = orc.seq_ppo_loss_grad(net, params, ro["obs"], ro["proprio"], ro["action"], ro["logp_old"], ro["value"], adv, ret, ro["done"], h0, c0,
                                      clip_eps=hp["clip_eps"], vclip_eps=hp["vclip_eps"], vf_coef=hp["vf_coef"], ent_coef=hp["ent_coef"])
    g = lrn.get_grads()
    bad = {n: rel_l2(g[a:b], qg[a:b]) for n, (a, b, _) in synth.param_slices(net).items() if rel_l2(g[a:b], qg[a:b]) > TOL_BF16}
    assert not bad, bad


@pytest.mark.parametrize("h,w,N,T", [(32, 32, 16, 8), (28, 31, 33, 4), (29, 42, 5, 3), (64, 64, 300, 4), (60, 89, 40, 4), (33, 65, 1100, 2)])
def test_small_network_convolutions(L, h, w, N, T):
    """Both convolutions of the small network in one kernel: odd sizes, ragged last pixels, fewer and more images than waves."""
    cfg = configs.get_config(0, num_envs=N, horizon=T)
    cfg["net"]["in_h"], cfg["net"]["in_w"] = h, w
    _check_gradients(L, cfg, N, T)

@pytest.mark.parametrize("h,w,views,P,N,T", [(32, 32, 2, 16, 9, 4), (33, 47, 3, 8, 5, 3), (60, 89, 2, 2056, 70, 4), (28, 31, 4, 2064, 3, 2), (64, 64, 2, 4096, 300, 2)])
def test_small_network_convolutions_of_several_views(L, h, w, views, P, N, T):
    """Views share a sample's proprioception, which is copied once, its first 2048 columns ahead of the rest."""
    cfg = configs.get_config(0, num_envs=N, horizon=T)
    cfg["net"].update(in_h=h, in_w=w, n_views=views, proprio_dim=P)
    _check_gradients(L, cfg, N, T)
    _check_forward(L, cfg, N, T)


@pytest.mark.parametrize("c0,conv,h,w,views,more", [(1, (16, 32), 33, 47, 2, {}), (1, (16, 32, 64, 128), 40, 72, 2, {}), (3, (32, 64, 64), 37, 53, 2, {}),
                                                    (3, (16, 32), 18, 66, 3, dict(embed_dim=24)), (1, (32, 64), 16, 130, 4, dict(embed_dim=32)),
                                                    (1, (8, 64, 128), 52, 60, 2, dict(embed_dim=16, layer_norm=0))])
def test_gradients_of_several_views_behind_layer_norm_or_embedding(L, c0, conv, h, w, views, more):
    """Strides between views in the unmasked transposed convolutions and the first layer's weight gradient from a stored one."""
    cfg = configs.get_config(1, num_envs=10, horizon=4)
    cfg["net"].update(dict(in_c=c0, in_h=h, in_w=w, n_views=views, conv_ch=list(conv), layer_norm=1), **more)
    _check_gradients(L, cfg, 10, 4)
    _check_forward(L, cfg, 10, 4)


@pytest.mark.parametrize("ci,hw", [(0, 28), (0, 60), (0, 64), (1, 64), (2, 120)])
def test_parameter_read_back(L, ci, hw):
    """Read-back of one piece (straight into the caller's memory), of two and five (staged by one thread) and of many (by four)."""
    net = configs.get_config(ci)["net"]
    net["in_h"] = net["in_w"] = hw
    params = synth.init_params(net, 2)
    lrn = L.Learner(net, 4, 1, "bf16")
    lrn.set_params(params)
    for _ in range(2):
        np.testing.assert_array_equal(lrn.get_params(), params)


@pytest.mark.parametrize("h,w", [(33, 41), (130, 70)])
def test_deepest_network_learns(L, h, w):
    """The largest number of weight re-packs a network may have: twelve transposed copies and, from the first backward
    pass on, two packed copies of seven convolutions.  Two updates, so that a step follows that pass."""
    cfg = configs.get_config(0, num_envs=6, horizon=4)
    net = cfg["net"]
    net.update(in_h=h, in_w=w, conv_ch=[8] * 8, fc_dim=[32, 16, 24, 16])
    import torch
    hp = dict(cfg["hp"], epochs=2, minibatches=1, seed=3, lr=1e-4)
    ro = synth.rollout(cfg, conditioned=True)
    params = synth.init_params(net, 9)
    a, b = (L.Learner(net, 6, 4, cfg["obs_dtype"]) for _ in range(2))
    for lrn in (a, b):
        lrn.set_params(params)
        fill_learner(lrn, cfg, ro)
        lrn.gae(torch.from_numpy(ro["last_value"]).cuda(), hp["gamma"], hp["lam"])
    a.update(hp)
    a.update(hp)
    # the same steps with fresh copies in front of every update
    b.update(hp)
    m, v, step, upd = b.get_opt_state()
    c = L.Learner(net, 6, 4, cfg["obs_dtype"])
    c.set_params(b.get_params())
    c.set_opt_state(m, v, step, upd)
    fill_learner(c, cfg, ro)
    c.gae(torch.from_numpy(ro["last_value"]).cuda(), hp["gamma"], hp["lam"])
    c.update(hp)
    np.testing.assert_array_equal(a.get_params(), c.get_params())
    assert np.abs(a.get_params() - params).max() > 1e-4


@pytest.mark.parametrize("h,w", [(40, 52), (72, 160), (120, 96)])
def test_gradient_sum_over_128_channels_is_rounded_once(L, h, w):
    """Transposed convolution from 128 gradient channels in a network with an embedding: channels 64 .. 127 carry the
    negative of channels 0 .. 63 but for 1/128, so that half-sums rounded to bf16 (2^-9 each) would leave the result
    with an error of about half of its own size, where one rounding leaves 2^-9."""
    cfg = configs.get_config(1, num_envs=10, horizon=4)
    net = cfg["net"]
    net.update(in_h=h, in_w=w, conv_ch=[16, 32, 64, 128], embed_dim=32)

    def opposed(params):
        sl = synth.param_slices(net)
        t = {n: params[a:b].reshape(s) for n, (a, b, s) in sl.items()}   # views
        t["conv3.w"][64:] = t["conv3.w"][:64]
        t["conv3.b"][64:] = t["conv3.b"][:64]
        e = t["emb.w"].reshape(32, 128, -1)
        e[:, :64] = np.sign(e[:, :64]) * 2.0 ** np.round(np.log2(np.abs(e[:, :64]) + 1e-6))   # both halves exact in bf16
        e[:, 64:] = -127 / 128 * e[:, :64]

    _check_gradients(L, cfg, 10, 4, opposed)


@pytest.mark.parametrize("conv,h,w", [((32, 64, 64, 128), 24, 200), ((32, 64, 64, 128), 61, 322), ((32, 64, 64, 128), 20, 380), ((64, 64, 128), 43, 170), ((32, 64, 64, 128), 20, 450)])
def test_gradient_sum_over_128_channels_of_wide_rows_is_rounded_once(L, conv, h, w):
    """The same sum in a feed-forward network whose layer before the last reads rows of more than 48 pixels of 64 channels: bands
    of fp32 halves up to the widest rows of the kernel (24 pixels of dY), and wider ones."""
    cfg = configs.get_config(1, num_envs=10, horizon=2)
    net, last = cfg["net"], f"conv{len(conv) - 1}"
    net.update(in_h=h, in_w=w, conv_ch=list(conv), fc_dim=[32])

    def opposed(params):
        sl = synth.param_slices(net)
        t = {n: params[a:b].reshape(s) for n, (a, b, s) in sl.items()}   # views
        t[last + ".w"][64:] = t[last + ".w"][:64]
        t[last + ".b"][64:] = t[last + ".b"][:64]
        f = t["fc0.w"][:, :-net["proprio_dim"]].reshape(32, 128, -1)     # a copy
        f[:, :64] = np.sign(f[:, :64]) * 2.0 ** np.round(np.log2(np.abs(f[:, :64]) + 1e-6))   # both halves exact in bf16
        f[:, 64:] = -127 / 128 * f[:, :64]
        t["fc0.w"][:, :-net["proprio_dim"]] = f.reshape(32, -1)

    _check_gradients(L, cfg, 10, 2, opposed)


@pytest.mark.parametrize("c0,conv,h,w", [(1, (32, 32), 60, 81), (1, (32, 64, 64), 64, 64), (3, (32, 64), 60, 80), (3, (32, 32), 60, 80),
                                         (3, (32, 16, 32), 45, 67), (3, (32, 32), 20, 270), (1, (32, 16), 24, 390)])
@pytest.mark.parametrize("spoil", [False, True])
def test_the_update_sees_the_policy_that_acted(L, c0, conv, h, w, spoil):
    """The first optimiser step on a fresh rollout evaluates the network as the policy step did, to the last bit (ratio 1 exactly),
    whichever kernels the two take: the first two layers in one kernel for both, or for the policy step alone (second layers of
    other than 64 channels).  With NaN in images too (spoil): the first layer rectifies its sums to 0, and they are those of the
    windows that hold it and no others."""
    import torch
    N, T = 128, 2
    cfg = configs.get_config(1, num_envs=N, horizon=T)
    net = cfg["net"]
    net.update(in_c=c0, in_h=h, in_w=w, conv_ch=list(conv), fc_dim=[64])
    params = synth.init_params(net, 9)
    a0, a1, _ = synth.param_slices(net)["logstd"]
    params[a0:a1] = -8.0   # the log-probability moves by 3000 times a change of the mean
    lrn = L.Learner(net, N, T, "bf16")
    lrn.set_params(params)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    for t in range(T):
        d = synth.rollout_step_torch(cfg, gen)
        obs = d["obs"].to(torch.bfloat16).contiguous()
        if spoil:
            obs[1::3, ..., h // 2, w // 3] = float("nan")
            obs[2::5, ..., 0, w - 1] = float("nan")
            obs[2::7, ..., h - 1, 0] = float("nan")
        lrn.act(t, obs, d["proprio"].contiguous(), torch.randn(N, net["act_dim"], generator=gen, device="cuda"))
        lrn.buffer_write_outcome(t, d["reward"].contiguous(), d["done"].contiguous())
    lrn.gae(torch.zeros(N, device="cuda"), 0.99, 0.95)
    st = lrn.update(dict(cfg["hp"], epochs=1, minibatches=1))
    assert st[0]["approx_kl"] == 0.0 and st[0]["clip_frac"] == 0.0


@pytest.mark.parametrize("h,w,hid,P,N,dtype", [(32, 32, 64, 32, 64, "fp32"), (16, 20, 32, 8, 3, "bf16"), (21, 27, 64, 16, 257, "fp32"), (40, 44, 64, 24, 130, "bf16"),
                                               (28, 33, 32, 40, 1024, "fp32"), (28, 28, 64, 32, 1025, "fp32"), (48, 48, 64, 32, 40, "fp32")])
def test_small_network_in_one_kernel(L, h, w, hid, P, N, dtype):
    """The small network's policy step and forward in one kernel (one to four samples per block, two depths of the hidden layer's slices,
    rows of any width and element offset) and, beyond its range, the separate launches: the sampled action against the oracle, the
    stored images and proprioception, and ratio 1 exactly in the update's first step."""
    import torch
    cfg = dict(configs.get_config(0, num_envs=N, horizon=2), obs_dtype=dtype)
    net = cfg["net"]
    net.update(in_h=h, in_w=w, fc_dim=[hid], proprio_dim=P)
    params = synth.init_params(net, 9)
    a0, a1, _ = synth.param_slices(net)["logstd"]
    params[a0:a1] = -8.0
    lrn = L.Learner(net, N, 2, dtype)
    lrn.set_params(params)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    odt = torch.float32 if dtype == "fp32" else torch.bfloat16
    for t in range(2):
        d = synth.rollout_step_torch(cfg, gen)
        room = torch.empty(d["obs"].numel() + 1, dtype=odt, device="cuda")   # the second step's images start at an odd element
        obs = room[t:t + d["obs"].numel()].view(d["obs"].shape)
        obs.copy_(d["obs"])
        pro, noise = d["proprio"].contiguous(), torch.randn(N, net["act_dim"], generator=gen, device="cuda")
        a, lp, v = lrn.act(t, obs, pro, noise)
        with orc.quant(1):
            oa, olp, ov = orc.act(net, params, obs.float().cpu().numpy(), pro.cpu().numpy(), noise.cpu().numpy())
        omu = oa - np.exp(-8.0) * noise.cpu().numpy()
        assert np.linalg.norm(a.cpu().numpy() - oa) <= TOL_BF16 * np.linalg.norm(omu) and rel_l2(v.cpu().numpy(), ov) <= TOL_BF16
        np.testing.assert_array_equal(lrn.buffer_read_obs(t).float().cpu().numpy(), obs.to(torch.bfloat16).float().cpu().numpy())
        lrn.buffer_write_outcome(t, d["reward"].contiguous(), d["done"].contiguous())
    mu, v2 = lrn.forward(torch.arange(N, 2 * N, device="cuda", dtype=torch.int32))   # the second step's
    assert rel_l2(mu.cpu().numpy(), omu) <= TOL_BF16 and torch.equal(v2, v)
    lrn.gae(torch.zeros(N, device="cuda"), 0.99, 0.95)
    st = lrn.update(dict(cfg["hp"], epochs=1, minibatches=2))
    assert st[0]["approx_kl"] == 0.0 and st[0]["clip_frac"] == 0.0


@pytest.mark.parametrize("where", ["proprio", "obs"])
def test_policy_step_into_the_memory_of_its_observations(L, where):
    """The C entry point takes the caller's output arrays, which may lie where the observations did: the small network's one kernel,
    in which a block may still read what another has written, is not the one that runs then."""
    import ctypes as C

    import torch
    N = 300
    cfg = configs.get_config(0, num_envs=N, horizon=1)
    net = cfg["net"]
    lrn = L.Learner(net, N, 1, "fp32")
    lrn.set_params(synth.init_params(net, 5))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    d = {k: v.contiguous() for k, v in synth.rollout_step_torch(cfg, gen).items()}
    noise = torch.randn(N, net["act_dim"], generator=gen, device="cuda")
    want = [x.clone() for x in lrn.act(0, d["obs"], d["proprio"], noise)]
    lrn.profile(True)
    lrn.act(0, d["obs"], d["proprio"], noise)
    assert "small_net_act" in lrn.profile_report()
    at = [1, 1 + noise.numel(), 1 + noise.numel() + N]   # the action from the second element on, log-probability and value behind it
    for use in ((0, 1, 2), (0,), (1,), (2,)):
        p = d["proprio"].clone() if where == "proprio" else d["proprio"]
        o = d["obs"].clone() if where == "obs" else d["obs"]
        room = (p if where == "proprio" else o).view(-1)
        out = [room[a:a + w.numel()] for a, w in zip(at, want)]
        ptr = [C.c_void_p(x.data_ptr()) if i in use else None for i, x in enumerate(out)]
        lrn.profile(True)
        lrn._chk(L._lib.ppo_act(lrn._h, 0, C.c_void_p(o.data_ptr()), C.c_void_p(p.data_ptr()), C.c_void_p(noise.data_ptr()), *ptr))
        torch.cuda.synchronize()
        assert "small_net_act" not in lrn.profile_report()
        for i in use:
            assert torch.equal(out[i].view(want[i].shape), want[i])


def test_read_back_staging_is_allocated_at_creation(L):
    """The first read of a context into memory in hand allocates nothing: its pinned staging (two pieces, 2 MiB, for this
    network) is part of ppo_create."""
    net = configs.get_config(1)["net"]
    params = synth.init_params(net, 2)
    out = np.zeros_like(params)

    def mapped():   # address space of the process, KiB
        with open("/proc/self/status") as f:
            return next(int(line.split()[1]) for line in f if line.startswith("VmSize"))

    grown = []
    keep = [L.Learner(net, 4, 1, "bf16") for _ in range(4)]
    for lrn in keep:
        lrn.set_params(params)
        before = mapped()
        assert L._lib.ppo_get_params(lrn._h, L._fp(out), out.size) == L.PPO_OK
        grown.append(mapped() - before)
        np.testing.assert_array_equal(out, params)
    assert min(grown) < 1024, grown   # (the runtime's own threads may map memory during any of them)


def test_read_back_behind_work_on_the_per_thread_stream(L):
    """hipStreamPerThread (handle 2) names another stream in every thread: what a read-back returns is ordered behind the
    update before it only if the thread that launched the update queues all of the read-back's transfers."""
    import types

    import torch
    cfg = configs.get_config(2, num_envs=64, horizon=4)
    net, hp = cfg["net"], dict(cfg["hp"], epochs=4, minibatches=2, seed=3)
    ro = synth.rollout(cfg, conditioned=True)
    params = synth.init_params(net, 9)
    dt = torch.float32 if cfg["obs_dtype"] == "fp32" else torch.bfloat16
    steps = [[torch.from_numpy(ro["obs"][t]).to("cuda", dt).contiguous()] +
             [torch.from_numpy(ro[k][t]).cuda().contiguous() for k in ("proprio", "action", "logp_old", "value", "reward", "done")] for t in range(4)]
    last = torch.from_numpy(ro["last_value"]).cuda()
    torch.cuda.synchronize()
    got = []
    for stream in (None, types.SimpleNamespace(cuda_stream=2, synchronize=torch.cuda.synchronize)):
        lrn = L.Learner(net, 64, 4, cfg["obs_dtype"], stream=stream)
        lrn.set_params(params)
        for t, d in enumerate(steps):
            lrn.buffer_write(t, *d)
        lrn.gae(last, hp["gamma"], hp["lam"])
        reads = []
        for _ in range(2):
            lrn.update(hp, want_stats=False)   # asynchronous
            reads.append(lrn.get_params())
        got.append(reads + [lrn.get_grads()] + list(lrn.get_opt_state()[:2]))
    assert got[0][0].size >= 8 << 18           # pieces for a team
    for x, y in zip(*got):
        np.testing.assert_array_equal(x, y)
    assert not np.array_equal(got[0][0], got[0][1])


def test_one_reduction_launch_per_step(L):
    """The partial sums of a backward pass of the full-size network (15 jobs at this batch) are taken by one launch."""
    import torch
    cfg = configs.get_config(2, num_envs=512, horizon=8)
    net, hp = cfg["net"], dict(cfg["hp"], epochs=3, minibatches=1, seed=3)
    lrn = L.Learner(net, 512, 8, "bf16")
    lrn.set_params(synth.init_params(net, 9))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1)
    keep = [synth.rollout_step_torch(cfg, gen) for _ in range(8)]
    for t, d in enumerate(keep):
        lrn.buffer_write(t, *(d[k].contiguous() for k in ("obs", "proprio", "action", "logp_old", "value", "reward", "done")))
    lrn.gae(torch.zeros(512, device="cuda"), hp["gamma"], hp["lam"])
    lrn.profile(True)
    lrn.update(hp)
    assert lrn.profile_report()["wgrad_reduce"]["launches"] == 3


@pytest.mark.parametrize("minibatches", [1, 2, 4])
@pytest.mark.parametrize("more", [{}, dict(layer_norm=1), dict(lstm_layers=1, lstm_units=64)])
def test_one_reduction_launch_per_step_of_a_small_network(L, more, minibatches):
    """The same for a network whose weight gradients are all cut into slices of 64 rows, at the largest chunk (1024 rows) and at
    fewer rows than the workspace was made for."""
    import torch
    cfg = configs.get_config(1, num_envs=256, horizon=4)
    net, hp = cfg["net"], dict(cfg["hp"], epochs=2, minibatches=minibatches, seed=3)
    net.update(dict(conv_ch=[8, 8], in_h=32, in_w=56, embed_dim=64, fc_dim=[64, 64], proprio_dim=8), **more)
    lrn = L.Learner(net, 256, 4, "bf16")
    lrn.set_params(synth.init_params(net, 9))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1)
    keep = [synth.rollout_step_torch(cfg, gen) for _ in range(4)]
    for t, d in enumerate(keep):
        lrn.buffer_write(t, *(d[k].contiguous() for k in ("obs", "proprio", "action", "logp_old", "value", "reward", "done")))
    lrn.gae(torch.zeros(256, device="cuda"), hp["gamma"], hp["lam"])
    lrn.profile(True)
    lrn.update(hp)
    assert lrn.profile_report()["wgrad_reduce"]["launches"] == 2 * minibatches


def test_memory_of_the_fused_first_layer(L):
    """The convolution in front of the first normalisation and its gradient stay in registers: a sample of a chunk takes the layer's
    rectified output, a gradient in either of two buffers and, of the second layer, three tensors, but not two more of the first's
    size."""
    import torch
    net = configs.get_config(1)["net"]
    net.update(in_h=120, in_w=160, conv_ch=[16, 32], layer_norm=1, fc_dim=[32])
    free = []
    for chunk in (256, 1280):
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        lrn = L.Learner(net, 1280, 1, "bf16", max_chunk=chunk)
        free.append(before - torch.cuda.mem_get_info()[0])
        lrn.close()
    first, second = 2 * 16 * 60 * 80, 2 * 32 * 30 * 40
    per_sample = (free[1] - free[0]) / 1024
    assert 3 * first + 3 * second <= per_sample <= 3.5 * first + 3 * second, per_sample / first
