"""GPU parity: the HIP library, called through its C ABI, against the CPU oracle on identical seeded inputs.

Tolerances (relative): 1e-5 on the fp32 accuracy path, 2e-2 on the bf16 MFMA path, for loss, u, g,
gradients and temperature gradients; scatter positions, untouched state entries and repeated runs are
compared bit for bit.
"""
import numpy as np
import pytest
import torch

from oracle import (ADAMW, LAMB, LION, SGDM, V0, V1, V2, V3, ema_update, fcco_step, gamma_cosine, normalize_rows,
                    temperature_update)
from paper_2407_01445_amd import binding as fc
from paper_2407_01445_amd.workloads import WORKLOADS, draw_indices, make_embeddings, round_to_bf16, step_seed

from gpu_harness import CANONICAL_FIELDS, DEV, RECORD_FILL, GpuStep, compare, rel_each, rel_inf, rel_l2

pytestmark = pytest.mark.gpu

TOL_F32 = 1e-5
TOL_BF16 = 2e-2


def oracle_step(g: GpuStep, img32, txt32, idx, u_img, u_txt, gamma, tau=0.07, tau_img=None, tau_txt=None):
    return fcco_step(img32.astype(np.float64), txt32.astype(np.float64), g.off, g.b, idx, u_img, u_txt,
                     version=g.version, gamma=gamma, eps=g.eps, rho=g.rho, tau=tau, tau_img=tau_img,
                     tau_txt=tau_txt, tau_grad_scale=g.scale)


def check_state(g: GpuStep, u_img_before, u_txt_before, idx, want_u_img, want_u_txt, tol):
    """Positions outside idx: bit-identical.  Positions in idx: equal to the dense u_new outputs bit for bit
    (the scatter wrote exactly what was reported) and within tol of the oracle."""
    ui, ut = g.u_img.cpu().numpy(), g.u_txt.cpu().numpy()
    mask = np.ones(g.N, bool)
    mask[idx] = False
    assert np.array_equal(ui[mask].view(np.uint32), u_img_before[mask].view(np.uint32))
    assert np.array_equal(ut[mask].view(np.uint32), u_txt_before[mask].view(np.uint32))
    assert np.array_equal(ui[idx], g.u_new_img.cpu().numpy())
    assert np.array_equal(ut[idx], g.u_new_txt.cpu().numpy())
    assert (ui[idx] > 0).all() and (ut[idx] > 0).all()
    assert rel_each(ui[idx], want_u_img[idx]) <= tol and rel_each(ut[idx], want_u_txt[idx]) <= tol


# ------------------------------------------------------------------------------- fp32 accuracy path
@pytest.mark.parametrize("version", [V1, V0, V3, V2])
def test_cfg0_ten_steps_f32(version):
    w = WORKLOADS["cfg0"]
    rho = {V1: 0.0, V0: 0.0, V3: 6.5, V2: 7.0}[version]
    g = GpuStep(B=w["B"], b=w["b"], off=0, d=w["d"], N=w["N"], dtype="f32", version=version, eps=w["eps"], rho=rho,
                tau=w["tau"], tau_grad_scale=1.0 / w["N"])
    u_img = np.zeros(w["N"])
    u_txt = np.zeros(w["N"])
    tau_arr = np.full(w["N"], np.float32(w["tau"]), np.float64)
    for step in range(w["steps"]):
        seed = step_seed("cfg0", step)
        img, txt = make_embeddings(seed, w["B"], w["d"], w["noise"], "f32")
        idx = draw_indices(seed + 500, w["b"], w["N"])
        before = (g.u_img.cpu().numpy(), g.u_txt.cpu().numpy())
        g.set_inputs(img, txt, idx)
        g.step(w["gamma"])
        want = oracle_step(g, img, txt, idx, u_img, u_txt, w["gamma"], tau=float(np.float32(w["tau"])),
                           tau_img=tau_arr, tau_txt=tau_arr)
        compare(g.outputs(), want, version, TOL_F32, "cfg0 v%d step %d" % (version, step))
        check_state(g, before[0], before[1], idx, u_img, u_txt, TOL_F32)


@pytest.mark.parametrize("version", [V0, V1, V2, V3])
def test_f32_ragged_strided_local_share(version):
    B, b, off, d, N = 37, 11, 13, 19, 200
    rng = np.random.default_rng(40 + version)
    img, txt = make_embeddings(91, B, d, 0.5, "f32")
    idx = draw_indices(92, b, N)
    u0i = np.where(rng.random(N) < 0.5, 0.0, rng.uniform(0.05, 2.0, N)).astype(np.float32)
    u0t = np.where(rng.random(N) < 0.5, 0.0, rng.uniform(0.05, 2.0, N)).astype(np.float32)
    t_img = rng.uniform(0.05, 0.1, N).astype(np.float32)
    t_txt = rng.uniform(0.05, 0.1, N).astype(np.float32)
    g = GpuStep(B=B, b=b, off=off, d=d, N=N, dtype="f32", version=version, eps=1e-3, rho=5.0, tau=0.07,
                tau_grad_scale=0.25, ld_img=24, ld_txt=19, u_img0=u0i, u_txt0=u0t, tau_img0=t_img, tau_txt0=t_txt)
    g.set_inputs(img, txt, idx)
    g.step(0.35)
    u_img, u_txt = u0i.astype(np.float64), u0t.astype(np.float64)
    want = oracle_step(g, img, txt, idx, u_img, u_txt, 0.35, tau=float(np.float32(0.07)),
                       tau_img=t_img.astype(np.float64), tau_txt=t_txt.astype(np.float64))
    compare(g.outputs(), want, version, TOL_F32, "f32 ragged v%d" % version)
    check_state(g, u0i, u0t, idx, u_img, u_txt, TOL_F32)


def test_f32_two_anchor_batch_and_gamma_one():
    """Smallest legal batch (B = 2) and gamma = 1: u must equal g exactly as reported."""
    img, txt = make_embeddings(5, 2, 8, 0.5, "f32")
    g = GpuStep(B=2, b=2, off=0, d=8, N=4, dtype="f32", version=V3, eps=1e-14, rho=6.5, tau=0.07,
                u_img0=np.array([0.5, 0, 0.25, 0], np.float32), u_txt0=np.array([0.5, 0, 0.25, 0], np.float32))
    idx = np.array([2, 1])
    g.set_inputs(img, txt, idx)
    g.step(1.0)
    u_img = np.array([0.5, 0, 0.25, 0])
    u_txt = u_img.copy()
    want = oracle_step(g, img, txt, idx, u_img, u_txt, 1.0, tau=float(np.float32(0.07)))
    compare(g.outputs(), want, V3, TOL_F32, "B=2")
    assert np.array_equal(g.u_new_img.cpu().numpy(), g.g_img.cpu().numpy())
    assert np.array_equal(g.u_new_txt.cpu().numpy(), g.g_txt.cpu().numpy())


F32_TILE_SHAPES = [
    # B, b, off, d, padding of the image rows
    (32, 32, 0, 8, 0),             # one whole tile, the whole batch local
    (33, 33, 0, 36, 4),            # one more row and column of tiles; a ragged last stage
    (66, 31, 34, 68, 0),           # two strips, tiles that end beyond the local anchors
    (130, 130, 0, 30, 1),          # rows that are not 16-byte aligned and end inside a word of four
    (300, 130, 170, 128, 0),       # several splits of the gradients' depth, the local range among them
    (4500, 70, 3, 36, 0),          # several contrast tiles behind one partial sum
    (1030, 1030, 0, 68, 0),        # 64 x 64 tiles, the whole batch local, ragged
    (2100, 550, 1201, 40, 4),      # 64 x 64 tiles, two strips, ragged
    # the last batches in plain loops, the first on tiles
    (16, 5, 9, 300, 0), (17, 5, 9, 300, 0), (24, 24, 0, 77, 1), (25, 25, 0, 77, 1), (24, 24, 0, 130, 0),
]


@pytest.mark.parametrize("B,b,off,d,pad", F32_TILE_SHAPES)
@pytest.mark.parametrize("version", [V0, V2, V3])
def test_f32_tiles_at_their_edges(B, b, off, d, pad, version):
    rng = np.random.default_rng(B + d + version)
    N = 6000
    img, txt = make_embeddings(B + 3, B, d, 0.5, "f32")
    idx = draw_indices(B + 4, b, N)
    u0i = np.where(rng.random(N) < 0.5, 0.0, rng.uniform(0.05, 2.0, N)).astype(np.float32)
    u0t = np.where(rng.random(N) < 0.5, 0.0, rng.uniform(0.05, 2.0, N)).astype(np.float32)
    t_img = rng.uniform(0.05, 0.1, N).astype(np.float32)
    t_txt = rng.uniform(0.05, 0.1, N).astype(np.float32)
    g = GpuStep(B=B, b=b, off=off, d=d, N=N, dtype="f32", version=version, eps=1e-6, rho=6.5, tau=0.07,
                tau_grad_scale=1.0 / N, ld_img=d + pad, u_img0=u0i, u_txt0=u0t, tau_img0=t_img, tau_txt0=t_txt)
    g.set_inputs(img, txt, idx)
    g.step(0.6)
    u_img, u_txt = u0i.astype(np.float64), u0t.astype(np.float64)
    want = oracle_step(g, img, txt, idx, u_img, u_txt, 0.6, tau=float(np.float32(0.07)), tau_img=t_img.astype(np.float64),
                       tau_txt=t_txt.astype(np.float64))
    first = g.outputs()
    compare(first, want, version, TOL_F32, "f32 tiles %s v%d" % ((B, b, off, d), version))
    check_state(g, u0i, u0t, idx, u_img, u_txt, TOL_F32)
    # whoever of several workgroups finishes a tile: the same bits (the state has moved on, so from the same state again)
    again = GpuStep(B=B, b=b, off=off, d=d, N=N, dtype="f32", version=version, eps=1e-6, rho=6.5, tau=0.07,
                    tau_grad_scale=1.0 / N, ld_img=d + pad, u_img0=u0i, u_txt0=u0t, tau_img0=t_img, tau_txt0=t_txt)
    again.set_inputs(img, txt, idx)
    again.step(0.6)
    assert all(np.array_equal(first[k], again.outputs()[k]) for k in ("d_img", "d_txt", "u_new_img", "u_new_txt"))


@pytest.mark.parametrize("B,b,off,d,pad", [
    # coefficients of 512 anchors in one pass and of more in two, the most that a workgroup forms, more than that; several
    # workgroups that finish anchors, the last one a single anchor; one anchor in all; 512 workgroups and more without them;
    # strips that prepare their anchors, of the widest rows with the whole batch local and of wide ragged ones without
    (448, 448, 0, 40, 0), (449, 449, 0, 40, 0), (900, 448, 450, 68, 4), (1024, 1024, 0, 20, 0), (1040, 1030, 5, 20, 4),
    (700, 257, 100, 300, 0), (65, 65, 0, 520, 0), (40, 1, 39, 36, 0), (520, 520, 0, 484, 0), (70, 70, 0, 512, 4),
    (140, 70, 31, 1030, 0)])
@pytest.mark.parametrize("version", [V0, V2, V3])
def test_f32_state_phase_inside_the_gradients(B, b, off, d, pad, version):
    test_f32_tiles_at_their_edges(B, b, off, d, pad, version)


@pytest.mark.parametrize("B,b,off,d,pad,nsplit,inside,prepares", [
    # a workgroup's coefficients: those of 512 anchors, one pass of its threads; of 576, two; of 1024 of the other side, the most; of
    # 1088, too many
    (448, 448, 0, 132, 0, 1, 1, 1), (449, 449, 0, 132, 4, 1, 1, 1), (1024, 1024, 0, 72, 0, 1, 1, 0), (1030, 1030, 0, 68, 4, 1, 0, 0),
    # 486 workgroups of the gradients with those that finish anchors, and 514
    (576, 576, 0, 404, 0, 1, 1, 1), (577, 577, 0, 404, 0, 1, 0, 1),
    # 24960 partial sums a workgroup, and 25792
    (1896, 948, 500, 20, 0, 4, 1, 0), (1930, 948, 500, 20, 0, 4, 0, 0),
    # strips that prepare: rows of 512 with the whole batch local, and wider; 512 workgroups, and with the whole batch local 529;
    # several contrast tiles behind one partial sum
    (96, 96, 0, 512, 0, 1, 1, 1), (96, 96, 0, 516, 0, 1, 1, 0), (2048, 128, 900, 36, 0, 9, 1, 1), (736, 736, 0, 40, 0, 2, 1, 0),
    (2100, 130, 1970, 36, 3, 9, 1, 1)])
def test_f32_launches_at_the_edges_of_their_rules(B, b, off, d, pad, nsplit, inside, prepares):
    """The plan, the launches that a timed step saw (a phase that no launch ran takes exactly 0), and the outputs."""
    version = V2 if B % 4 else V3
    g = GpuStep(B=B, b=b, off=off, d=d, N=6000, dtype="f32", version=version, eps=1e-6, rho=6.5, tau=0.07, ld_img=d + pad)
    plan = fc.fastclip_describe(g.config(0.6))
    assert (plan["tile"], plan["nsplit"], plan["fused_state"]) == (0, nsplit, inside)
    test_f32_tiles_at_their_edges(B, b, off, d, pad, version)
    img, txt = make_embeddings(B + 3, B, d, 0.5, "f32")
    g.set_inputs(img, txt, draw_indices(B + 4, b, 6000))
    phases = g.step(0.6, timed=True)
    assert [phases[k] > 0.0 for k in ("prep", "strips", "state", "finalize")] == [not prepares, True, not inside, True], phases


@pytest.mark.parametrize("version", [V0, V2])
def test_f32_gathered_state_on_several_tiles(version):
    run_gathered(300, 130, 170, 72, version, "f32", TOL_F32)


@pytest.mark.parametrize("version", [V0, V2])
def test_f32_gathered_state_on_few_pairs(version):
    run_gathered(23, 6, 11, 70, version, "f32", TOL_F32, N=200, ld_pad=3)


# Two draws of a 400-case random sweep of the fp32 path on which the loss nearly cancels (case A: tau mean(log) = -0.911
# against 2 rho tau = +0.910; case B: 112 logarithms of values around 1 whose mean is 0.0035 against a mean magnitude
# of 3.2).  An error relative to the loss itself reads 700 - 900 times the error of the terms there; relative to the
# terms' magnitudes (the metric of compare()) these draws are like any other.  The fp32 path forms its logarithms and
# the sums behind the scalars in fp64; what is left is the fp32 rounding of the stored state u^{t+1} itself (1e-7
# relative, hence 1e-7 absolute in log u, times tau), which no arithmetic after it can take back: relative to the
# loss itself the two draws then read 1e-5 and 3e-6 (3.4e-5 and 2.6e-5 with fp32 logarithms and partial sums).
CANCELLING_LOSS_DRAWS = [
    # case, B, b, off, d, version, gathered, gamma, N, ld padding of img
    (304, 4, 1, 1, 5, V3, True, 1.0, 2, 3),
    (378, 76, 56, 20, 2, V1, False, 0.25, 108, 8),
]


@pytest.mark.parametrize("case,B,b,off,d,version,gathered,gamma,N,pad", CANCELLING_LOSS_DRAWS)
def test_f32_draws_whose_loss_terms_cancel(case, B, b, off, d, version, gathered, gamma, N, pad):
    rng = np.random.default_rng(case + 31000)
    img, txt = make_embeddings(case + 7, B, d, 0.5, "f32")
    idx = draw_indices(case + 3, b, N)
    u0i = np.where(rng.random(N) < 0.5, 0.0, rng.uniform(0.05, 2.0, N)).astype(np.float32)
    u0t = np.where(rng.random(N) < 0.5, 0.0, rng.uniform(0.05, 2.0, N)).astype(np.float32)
    t_img = rng.uniform(0.05, 0.1, N).astype(np.float32)
    t_txt = rng.uniform(0.05, 0.1, N).astype(np.float32)
    f64 = lambda a: None if a is None else a.astype(np.float64)
    gath, extra = None, {}
    if gathered:
        ug1 = rng.uniform(0.05, 2.0, B).astype(np.float32)
        ug2 = rng.uniform(0.05, 2.0, B).astype(np.float32)
        gath = dict(u_img=ug1, u_txt=ug2, tau_img=None, tau_txt=None)
        extra = dict(u_glob_img=f64(ug1), u_glob_txt=f64(ug2))
    g = GpuStep(B=B, b=b, off=off, d=d, N=N, dtype="f32", version=version, eps=1e-6, rho=6.5, tau=0.07,
                tau_grad_scale=1.0 / N, ld_img=d + pad, ld_txt=d + 8, u_img0=u0i, u_txt0=u0t, tau_img0=t_img,
                tau_txt0=t_txt, gathered=gath)
    g.set_inputs(img, txt, idx)
    g.step(gamma)
    u_img, u_txt = u0i.astype(np.float64), u0t.astype(np.float64)
    want = fcco_step(img.astype(np.float64), txt.astype(np.float64), off, b, idx, u_img, u_txt, version=version,
                     gamma=gamma, eps=g.eps, rho=g.rho, tau=float(np.float32(0.07)), tau_img=f64(t_img),
                     tau_txt=f64(t_txt), tau_grad_scale=g.scale, **extra)
    assert want["loss_abs"] > 500 * abs(want["loss"])          # the draw is what the comment says it is
    compare(g.outputs(), want, version, TOL_F32, "cancelling loss, draw %d" % case)


# ------------------------------------------------------------------------------- the method's own operating range
def trained_like_embeddings(seed, B, d, dtype):
    """Pairs as a trained model produces them: text = normalise(image + small noise), s_ii about 0.9."""
    return make_embeddings(seed, B, d, 0.48 / np.sqrt(d), dtype)


def small_history(rng, N):
    """State of a trained model's scale (g about exp(-0.9 / tau)): half never visited, the rest 1e-13 .. 1e-4."""
    u = np.exp(rng.uniform(np.log(1e-13), np.log(1e-4), N))
    return np.where(rng.random(N) < 0.5, 0.0, u).astype(np.float32)


@pytest.mark.parametrize("dtype,tol,shape", [("f32", TOL_F32, (37, 11, 13, 19)), ("f32", TOL_F32, (64, 64, 0, 32)),
                                             ("bf16", TOL_BF16, (700, 300, 133, 72)),
                                             ("bf16", TOL_BF16, (1024, 320, 704, 128)),
                                             ("bf16", TOL_BF16, (768, 768, 0, 192))])
@pytest.mark.parametrize("tau", [0.03, 0.025])
@pytest.mark.parametrize("version", [V0, V2, V3])
@pytest.mark.parametrize("trained", [False, True])
def test_small_temperatures_and_trained_statistics(dtype, tol, shape, tau, version, trained):
    """Temperatures at and below the value where the paper drops the temperature's learning rate (0.03; the documented
    domain ends at 0.023), global and per sample, on early-training pairs and on pairs with s_ii about 0.9, where g is
    about exp(-0.9 / tau) = 1e-13 .. 1e-16, eps = 1e-14 matters, and the coefficients 1 / (eps + u) are 1e10 and more."""
    B, b, off, d = shape
    N = 3000
    rng = np.random.default_rng(int(1000 * tau) + 10 * version + B)
    img, txt = (trained_like_embeddings if trained else lambda s, B, d, t: make_embeddings(s, B, d, 0.5, t))(B + 41, B, d, dtype)
    idx = draw_indices(B + 42, b, N)
    if trained:
        u0i, u0t = small_history(rng, N), small_history(rng, N)
    else:
        u0i = np.where(rng.random(N) < 0.5, 0.0, rng.uniform(0.05, 2.0, N)).astype(np.float32)
        u0t = np.where(rng.random(N) < 0.5, 0.0, rng.uniform(0.05, 2.0, N)).astype(np.float32)
    # per-sample temperatures around tau, none below the documented 0.023
    t_img = rng.uniform(max(0.0235, 0.9 * tau), 1.3 * tau, N).astype(np.float32)
    t_txt = rng.uniform(max(0.0235, 0.9 * tau), 1.3 * tau, N).astype(np.float32)
    g = GpuStep(B=B, b=b, off=off, d=d, N=N, dtype=dtype, version=version, eps=1e-14, rho=6.5, tau=tau,
                tau_grad_scale=1.0 / N, u_img0=u0i, u_txt0=u0t, tau_img0=t_img, tau_txt0=t_txt)
    g.set_inputs(img, txt, idx)
    g.step(0.6)
    u_img, u_txt = u0i.astype(np.float64), u0t.astype(np.float64)
    want = oracle_step(g, img, txt, idx, u_img, u_txt, 0.6, tau=float(np.float32(tau)),
                       tau_img=t_img.astype(np.float64), tau_txt=t_txt.astype(np.float64))
    if trained:
        assert np.median(want["g_img"]) < 1e-6
    compare(g.outputs(), want, version, tol, "tau %.3f %s %s %s v%d" % (tau, "trained" if trained else "early", dtype,
                                                                      shape, version))
    check_state(g, u0i, u0t, idx, u_img, u_txt, tol)


# ------------------------------------------------------------------------------- bf16 MFMA path, small shapes
BF16_SMALL = [
    # B, b, off, d: several 256-tiles with ragged tails in anchors, contrasts and width; local share and full batch
    (700, 300, 133, 72),
    (520, 520, 0, 64),
    (1000, 64, 936, 136),
    (257, 257, 0, 8),
    # whole 256-tiles (the unguarded persistent kernels) next to ragged ones, widths that are whole / ragged stages
    (768, 512, 256, 128),
    (1024, 300, 512, 256),
    (900, 512, 388, 96),
    # fewer local anchors than a tile has rows: the persistent kernel computes on the global rows that follow them
    # (its results for those land in padding); a last anchor tile that would run past the global batch is guarded
    (768, 100, 300, 128),
    (1024, 300, 724, 256),
    # ... and 320 anchors at the very end of the global batch: the last tile is moved back to end at b and recomputes
    # 192 anchors of the first one
    (1024, 320, 704, 128),
    # enough contrast columns for a split contraction and an anchor count that is no multiple of 4: the last group of
    # four rows of the split partial sums is ragged where the wavefronts of a block share the splits
    (1100, 203, 50, 136),
    # wide embeddings: many 64-deep stages per tile, a width of whole stages and one with a ragged last stage
    (700, 300, 133, 2048),
    (300, 300, 0, 4104),
    # the whole batch local and only whole tiles
    (512, 512, 0, 128),
    (768, 768, 0, 192),
    # ... and more tiles than compute units: the similarity matrix is formed once, sums down the columns
    (3072, 3072, 0, 128),
]


@pytest.mark.parametrize("B,b,off,d", BF16_SMALL)
@pytest.mark.parametrize("version", [V0, V1, V2, V3])
def test_bf16_small_shapes(B, b, off, d, version):
    N = 5000
    rng = np.random.default_rng(B + version)
    img, txt = make_embeddings(B + d, B, d, 0.5, "bf16")
    idx = draw_indices(B + 1, b, N)
    u0i = np.where(rng.random(N) < 0.5, 0.0, rng.uniform(0.05, 2.0, N)).astype(np.float32)
    u0t = np.where(rng.random(N) < 0.5, 0.0, rng.uniform(0.05, 2.0, N)).astype(np.float32)
    t_img = rng.uniform(0.05, 0.1, N).astype(np.float32)
    t_txt = rng.uniform(0.05, 0.1, N).astype(np.float32)
    g = GpuStep(B=B, b=b, off=off, d=d, N=N, dtype="bf16", version=version, eps=1e-6, rho=6.5, tau=0.07,
                tau_grad_scale=1.0 / N, ld_img=d + 8, ld_txt=d, u_img0=u0i, u_txt0=u0t, tau_img0=t_img, tau_txt0=t_txt)
    g.set_inputs(img, txt, idx)
    g.step(0.6)
    u_img, u_txt = u0i.astype(np.float64), u0t.astype(np.float64)
    want = oracle_step(g, img, txt, idx, u_img, u_txt, 0.6, tau=float(np.float32(0.07)),
                       tau_img=t_img.astype(np.float64), tau_txt=t_txt.astype(np.float64))
    compare(g.outputs(), want, version, TOL_BF16, "bf16 %s v%d" % ((B, b, off, d), version))
    check_state(g, u0i, u0t, idx, u_img, u_txt, TOL_BF16)


SINGLE_PASS_SHAPES = [
    # b == B, off == 0, ragged in anchors / contrasts / width: every tile is guarded
    (520, 520, 64), (1000, 1000, 136), (257, 257, 8), (300, 300, 72), (40, 40, 16),
    # whole tiles only (the persistent kernel alone), forced below the size at which the library chooses the mode
    (768, 768, 192), (512, 512, 128),
    # whole tiles of the persistent kernel next to guarded ones (ragged last row and column of tiles)
    (900, 900, 128), (1100, 1100, 256),
]


@pytest.mark.parametrize("B,b,d", SINGLE_PASS_SHAPES)
@pytest.mark.parametrize("version", [V0, V1, V2, V3])
def test_bf16_single_similarity_pass_on_any_shape(B, b, d, version):
    """FASTCLIP_SINGLE_PASS: with the whole batch local the similarity matrix is formed once (the text strip is the
    transpose of the image strip), also where tiles are ragged: against the oracle, and close to the two-strip form."""
    N = 5000
    rng = np.random.default_rng(B + 7 * version)
    img, txt = make_embeddings(B + d + 1, B, d, 0.5, "bf16")
    idx = draw_indices(B + 2, b, N)
    u0i = np.where(rng.random(N) < 0.5, 0.0, rng.uniform(0.05, 2.0, N)).astype(np.float32)
    u0t = np.where(rng.random(N) < 0.5, 0.0, rng.uniform(0.05, 2.0, N)).astype(np.float32)
    t_img = rng.uniform(0.05, 0.1, N).astype(np.float32)
    t_txt = rng.uniform(0.05, 0.1, N).astype(np.float32)
    outs = []
    for single in (True, False):
        g = GpuStep(B=B, b=b, off=0, d=d, N=N, dtype="bf16", version=version, eps=1e-6, rho=6.5, tau=0.07,
                    tau_grad_scale=1.0 / N, ld_img=d, ld_txt=d + 8, u_img0=u0i, u_txt0=u0t, tau_img0=t_img,
                    tau_txt0=t_txt, single_pass=single)
        g.set_inputs(img, txt, idx)
        g.step(0.6)
        u_img, u_txt = u0i.astype(np.float64), u0t.astype(np.float64)
        want = oracle_step(g, img, txt, idx, u_img, u_txt, 0.6, tau=float(np.float32(0.07)),
                           tau_img=t_img.astype(np.float64), tau_txt=t_txt.astype(np.float64))
        compare(g.outputs(), want, version, TOL_BF16, "bf16 single pass %s %s v%d" % (single, (B, b, d), version))
        check_state(g, u0i, u0t, idx, u_img, u_txt, TOL_BF16)
        outs.append(g.outputs())
    # the two forms round the same dot products: sums differ in their order only
    for k in ("g_img", "g_txt", "u_new_img", "u_new_txt"):
        assert rel_each(outs[0][k], outs[1][k]) < 1e-4, k


@pytest.mark.parametrize("B,b,d", [
    # (The weights are two strips, w / c of either side, and each is read by rows.  The shapes are those at which one strip read both
    # ways could go wrong:)
    # one strip of weights read by rows and by columns: columns of a tile of rows that the strip does not have, a last stage of one
    # row, several splits, output tiles of either width
    (257, 257, 8), (320, 320, 200), (449, 449, 264), (1217, 1217, 136), (2300, 2300, 72)])
def test_bf16_single_similarity_pass_contracts_one_strip_both_ways(B, b, d):
    test_bf16_single_similarity_pass_on_any_shape(B, b, d, V2 if B % 2 else V3)


def test_bf16_single_similarity_pass_chosen_by_the_library_on_a_ragged_batch():
    """3000 x 3000 pairs: more 256 x 256 tiles than compute units, so the library forms the similarity matrix once without
    being asked; 11 x 11 whole tiles go to the persistent kernel, the ragged last row and column to the guarded one."""
    B = b = 3000
    d, N = 128, 20_000
    rng = np.random.default_rng(77)
    img, txt = make_embeddings(78, B, d, 0.5, "bf16")
    idx = draw_indices(79, b, N)
    u0i = np.where(rng.random(N) < 0.5, 0.0, rng.uniform(0.05, 2.0, N)).astype(np.float32)
    u0t = np.where(rng.random(N) < 0.5, 0.0, rng.uniform(0.05, 2.0, N)).astype(np.float32)
    t_img = rng.uniform(0.05, 0.1, N).astype(np.float32)
    t_txt = rng.uniform(0.05, 0.1, N).astype(np.float32)
    g = GpuStep(B=B, b=b, off=0, d=d, N=N, dtype="bf16", version=V2, eps=1e-6, rho=6.5, tau=0.07,
                tau_grad_scale=1.0 / N, u_img0=u0i, u_txt0=u0t, tau_img0=t_img, tau_txt0=t_txt)
    g.set_inputs(img, txt, idx)
    g.step(0.6)
    u_img, u_txt = u0i.astype(np.float64), u0t.astype(np.float64)
    want = oracle_step(g, img, txt, idx, u_img, u_txt, 0.6, tau=0.07, tau_img=t_img.astype(np.float64),
                       tau_txt=t_txt.astype(np.float64))
    compare(g.outputs(), want, V2, TOL_BF16, "bf16 single pass 3000", tol_measured=TOL_BF16_MEASURED)
    check_state(g, u0i, u0t, idx, u_img, u_txt, TOL_BF16)


TILES_128_SHAPES = [
    # ragged in anchors, contrasts and width; a width below one stage; the whole batch local
    (700, 300, 133, 72), (520, 520, 0, 64), (1000, 64, 936, 136), (257, 257, 0, 8),
    # whole stages and tiles next to ragged ones; anchors at the very end of the global batch
    (768, 512, 256, 128), (1024, 300, 724, 256), (1024, 320, 704, 128), (1100, 203, 50, 136),
    # wide rows: many stages per tile, one width with a ragged last stage
    (700, 300, 133, 2048), (300, 300, 0, 4104),
    # the paper's own per-GPU shapes (128 - 640 anchors of 1024 - 5120, width 512) and the two small workloads' shapes
    (1024, 128, 128, 512), (2560, 320, 320, 512), (5120, 640, 640, 512), (1024, 1024, 0, 512), (8192, 256, 1280, 512),
]


@pytest.mark.parametrize("B,b,off,d", TILES_128_SHAPES)
@pytest.mark.parametrize("version", [V0, V1, V2, V3])
def test_bf16_tiles_128(B, b, off, d, version):
    """FASTCLIP_TILES_128: strips and contraction on 128 x 128 tiles (four times the workgroups, output tiles finished in
    place when the column range needs no split), against the oracle and close to the default path."""
    N = 5000
    rng = np.random.default_rng(B + 3 * version)
    img, txt = make_embeddings(B + d + 5, B, d, 0.5, "bf16")
    idx = draw_indices(B + 6, b, N)
    u0i = np.where(rng.random(N) < 0.5, 0.0, rng.uniform(0.05, 2.0, N)).astype(np.float32)
    u0t = np.where(rng.random(N) < 0.5, 0.0, rng.uniform(0.05, 2.0, N)).astype(np.float32)
    t_img = rng.uniform(0.05, 0.1, N).astype(np.float32)
    t_txt = rng.uniform(0.05, 0.1, N).astype(np.float32)
    u_img, u_txt = u0i.astype(np.float64), u0t.astype(np.float64)
    want = None
    outs = []
    for small in (True, False):
        print("[tiles 128 = %s] %s v%d" % (small, (B, b, off, d), version), flush=True)
        g = GpuStep(B=B, b=b, off=off, d=d, N=N, dtype="bf16", version=version, eps=1e-6, rho=6.5, tau=0.07,
                    tau_grad_scale=1.0 / N, ld_img=d + 8, ld_txt=d, u_img0=u0i, u_txt0=u0t, tau_img0=t_img, tau_txt0=t_txt,
                    tiles=128 if small else 256)
        g.set_inputs(img, txt, idx)
        g.step(0.6)
        if want is None:
            want = oracle_step(g, img, txt, idx, u_img, u_txt, 0.6, tau=float(np.float32(0.07)),
                               tau_img=t_img.astype(np.float64), tau_txt=t_txt.astype(np.float64))
        compare(g.outputs(), want, version, TOL_BF16, "bf16 tiles 128 %s %s v%d" % (small, (B, b, off, d), version))
        check_state(g, u0i, u0t, idx, u_img, u_txt, TOL_BF16)
        outs.append(g.outputs())
    for k in ("g_img", "g_txt", "u_new_img", "u_new_txt"):      # the same exponentials, summed in another order
        assert rel_each(outs[0][k], outs[1][k]) < 1e-4, k


@pytest.mark.parametrize("B,b,off,d", [
    # fewer rows than a stage is deep, the columns' numbering wrapping inside it; one stage more or less; a last row block of one
    (7, 3, 2, 8), (16, 16, 0, 64), (17, 9, 8, 72), (129, 65, 64, 520),
    # four groups of 256 local anchors, of three splits or one, on 128-row output tiles too
    (2048, 2048, 0, 64), (4000, 1000, 3000, 760), (1030, 1023, 7, 1016),
    # the depth split over eight workgroups
    (8192, 64, 8128, 64),
    # contraction on 128 x 128 output tiles behind the fold: ragged everywhere, one split; rows that are not the first, a
    # last row block of one; two splits, strips of two workgroups per compute unit with a guarded last stage
    (900, 900, 0, 2072), (1100, 897, 133, 2072), (1450, 1400, 33, 808)])
def test_bf16_tiles_128_edges(B, b, off, d):
    """The shapes at which the kernels of the 128 x 128-tile path change what they do, as in test_bf16_tiles_128."""
    test_bf16_tiles_128(B, b, off, d, V2 if B % 2 else V3)


def test_calls_without_a_stream_take_the_current_one():
    """On torch's default stream, on a stream of the program's own and back, as torch.cuda.current_stream() names them."""
    side = torch.cuda.Stream()
    for context in (None, side, None):
        with torch.cuda.stream(context):
            assert fc._stream(None) == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(side):
        assert fc._stream(None) == side.cuda_stream and fc._stream(torch.cuda.default_stream()) == torch.cuda.default_stream().cuda_stream


@pytest.mark.parametrize("B,b,off,d", [
    # strip tiles of 32 anchors up to one round of them, then of 64 and of 128; with a last anchor alone in its tile; one step and
    # a half; rows that the strips prepare and, wider, the launch before them
    (2048, 256, 768, 512), (2048, 257, 700, 512), (2049, 256, 1000, 264), (1000, 97, 500, 192), (1100, 33, 1000, 136),
    (600, 290, 10, 1200), (600, 290, 10, 1208)])
def test_bf16_small_tiles_of_32_anchors(B, b, off, d):
    test_bf16_tiles_128(B, b, off, d, V2 if d % 3 else V3)


@pytest.mark.parametrize("B,b,off,d,fused,nsplit", [
    # 32 x 32 output tiles: one stage, one row, widths inside a tile
    (33, 33, 0, 8, 1, 1), (40, 1, 39, 40, 1, 1), (65, 31, 34, 24, 1, 1),
    (300, 256, 40, 512, 1, 1), (257, 255, 2, 504, 1, 1),     # ... on every compute unit: the anchors finished by the first columns
    (1100, 130, 700, 200, 1, 1),                             # ... several stages per wave, rows that wrap around the batch
    # coefficients of several groups of 256 local anchors, which the waves share out: three groups; five, of two in a split;
    # five and eight in one workgroup (64-row tiles), six (128-row tiles) and, with a second pass, nine
    (700, 600, 60, 256, 1, 1), (1300, 1030, 270, 128, 1, 3), (1300, 1270, 30, 256, 1, 1), (2048, 2000, 40, 192, 1, 1),
    (1600, 1500, 33, 512, 1, 1), (2300, 2250, 30, 448, 1, 1),
    (2304, 1000, 1200, 760, 1, 1), (3000, 520, 100, 72, 1, 6),   # 128-row tiles; anchors of several finishing workgroups, splits
    (300, 300, 0, 4104, 0, 1)])                              # several rounds of workgroups: the state phase on its own
def test_bf16_small_tile_plans(B, b, off, d, fused, nsplit):
    """The plans of the small tiles at the sizes where they change what they do (tile size, who forms the coefficients and who
    finishes the anchors, groups and slices of the partial sums), as in test_bf16_tiles_128."""
    plan = fc.fastclip_describe(fc.make_config(version=V3, emb_dtype=fc.BF16, B=B, b=b, off=off, d=d, N=5000, gamma=0.6,
                                               eps=1e-6, rho=6.5, ld_img=d + 8, ld_txt=d, flags=fc.TILES_128))
    assert (plan["tile"], plan["fused_state"], plan["nsplit"]) == (128, fused, nsplit)
    test_bf16_tiles_128(B, b, off, d, V2 if d % 3 else V3)


@pytest.mark.parametrize("B,b,off,d", [
    (256, 200, 56, 8), (1056, 300, 700, 192), (1040, 257, 100, 200), (1056, 256, 800, 256),     # one or two tiles of columns,
    (2056, 300, 0, 384), (1100, 600, 500, 392), (1300, 260, 1040, 512), (900, 900, 0, 520),      # whole ones and the first words
    (700, 513, 100, 768)])                                                                       # of another; ragged depths
def test_bf16_large_tile_output_columns(B, b, off, d):
    """Output tiles of 192 and of 256 columns in the contraction of the large tiles, as in test_bf16_tiles_128 (which runs the
    batch on the large tiles too)."""
    test_bf16_tiles_128(B, b, off, d, V2 if d % 3 else V3)


@pytest.mark.parametrize("B,b,off,d", BF16_SMALL[:-1] + [(1024, 128, 128, 512), (2560, 320, 320, 512), (5120, 640, 640, 512)])
@pytest.mark.parametrize("version", [V0, V1, V2, V3])
def test_bf16_fine_tiles(B, b, off, d, version):
    """The opt-in fine-tile path (128 x 128 strip tiles, 64 x 64 output tiles finished in place) on the small shapes
    and on the paper's own per-GPU shapes, against the oracle."""
    N = 5000
    rng = np.random.default_rng(B + version)
    img, txt = make_embeddings(B + d, B, d, 0.5, "bf16")
    idx = draw_indices(B + 1, b, N)
    u0i = np.where(rng.random(N) < 0.5, 0.0, rng.uniform(0.05, 2.0, N)).astype(np.float32)
    u0t = np.where(rng.random(N) < 0.5, 0.0, rng.uniform(0.05, 2.0, N)).astype(np.float32)
    t_img = rng.uniform(0.05, 0.1, N).astype(np.float32)
    t_txt = rng.uniform(0.05, 0.1, N).astype(np.float32)
    g = GpuStep(B=B, b=b, off=off, d=d, N=N, dtype="bf16", version=version, eps=1e-6, rho=6.5, tau=0.07,
                tau_grad_scale=1.0 / N, ld_img=d + 8, ld_txt=d, u_img0=u0i, u_txt0=u0t, tau_img0=t_img, tau_txt0=t_txt,
                fine_tiles=True)
    g.set_inputs(img, txt, idx)
    g.step(0.6)
    u_img, u_txt = u0i.astype(np.float64), u0t.astype(np.float64)
    want = oracle_step(g, img, txt, idx, u_img, u_txt, 0.6, tau=float(np.float32(0.07)),
                       tau_img=t_img.astype(np.float64), tau_txt=t_txt.astype(np.float64))
    compare(g.outputs(), want, version, TOL_BF16, "bf16 fine tiles %s v%d" % ((B, b, off, d), version))
    check_state(g, u0i, u0t, idx, u_img, u_txt, TOL_BF16)


def test_bf16_large_ragged_global_batch():
    """One worker's 256 anchors against 40003 global pairs: two strips of 156 whole contrast tiles plus a ragged last
    one, 1251 contraction stages split over the column range."""
    B, b, off, d, N = 40_003, 256, 20_096, 128, 50_000
    img, txt = make_embeddings(91, B, d, 0.5, "bf16")
    idx = draw_indices(92, b, N)
    g = GpuStep(B=B, b=b, off=off, d=d, N=N, dtype="bf16", version=V3, eps=1e-14, rho=8.5, tau=0.07)
    g.set_inputs(img, txt, idx)
    g.step(0.9)
    u_img, u_txt = np.zeros(N), np.zeros(N)
    want = oracle_step(g, img, txt, idx, u_img, u_txt, 0.9, tau=float(np.float32(0.07)))
    compare(g.outputs(), want, V3, TOL_BF16, "bf16 large B")
    check_state(g, np.zeros(N, np.float32), np.zeros(N, np.float32), idx, u_img, u_txt, TOL_BF16)


def test_bf16_repeatable_bit_for_bit():
    B, b, off, d, N = 700, 300, 133, 72, 5000
    img, txt = make_embeddings(3, B, d, 0.5, "bf16")
    idx = draw_indices(4, b, N)
    res = []
    for _ in range(2):
        g = GpuStep(B=B, b=b, off=off, d=d, N=N, dtype="bf16", version=V3, eps=1e-14, rho=6.5)
        g.set_inputs(img, txt, idx)
        g.step(0.7)
        res.append((g.d_img.cpu(), g.d_txt.cpu(), g.u_img.cpu(), g.loss.cpu(), g.d_tau.cpu()))
    for x, y in zip(*res):
        assert torch.equal(x, y)


# ------------------------------------------------------------------------------- gathered state (Eqs. 3/5/7 in full)
def gathered_inputs(rng, B, version):
    """What the other workers report: u^{t+1} of every global row, and for V2 the rows' temperatures; the entries
    of the local rows are poison on the GPU side (they must not be read) and arbitrary on the oracle side."""
    ug1 = rng.uniform(0.05, 2.0, B).astype(np.float32)
    ug2 = rng.uniform(0.05, 2.0, B).astype(np.float32)
    tg1 = rng.uniform(0.05, 0.1, B).astype(np.float32) if version == V2 else None
    tg2 = rng.uniform(0.05, 0.1, B).astype(np.float32) if version == V2 else None
    return ug1, ug2, tg1, tg2


def run_gathered(B, b, off, d, version, dtype, tol, N=5000, ld_pad=0, tiles=256):
    rng = np.random.default_rng(7 * B + version)
    img, txt = make_embeddings(B + d + 1, B, d, 0.5, dtype)
    idx = draw_indices(B + 2, b, N)
    u0i = np.where(rng.random(N) < 0.5, 0.0, rng.uniform(0.05, 2.0, N)).astype(np.float32)
    u0t = np.where(rng.random(N) < 0.5, 0.0, rng.uniform(0.05, 2.0, N)).astype(np.float32)
    t_img = rng.uniform(0.05, 0.1, N).astype(np.float32)
    t_txt = rng.uniform(0.05, 0.1, N).astype(np.float32)
    ug1, ug2, tg1, tg2 = gathered_inputs(rng, B, version)

    def poisoned(a):
        if a is None:
            return None
        a = a.copy()
        a[off:off + b] = np.nan
        return a
    g = GpuStep(B=B, b=b, off=off, d=d, N=N, dtype=dtype, version=version, eps=1e-6, rho=6.5, tau=0.07,
                tau_grad_scale=1.0 / N, ld_img=d + ld_pad, ld_txt=d, u_img0=u0i, u_txt0=u0t, tau_img0=t_img,
                tau_txt0=t_txt, gathered=dict(u_img=poisoned(ug1), u_txt=poisoned(ug2), tau_img=poisoned(tg1),
                                              tau_txt=poisoned(tg2)), tiles=tiles)
    g.set_inputs(img, txt, idx)
    g.step(0.6)
    u_img, u_txt = u0i.astype(np.float64), u0t.astype(np.float64)
    f64 = lambda a: None if a is None else a.astype(np.float64)
    want = fcco_step(img.astype(np.float64), txt.astype(np.float64), off, b, idx, u_img, u_txt, version=version,
                     gamma=0.6, eps=g.eps, rho=g.rho, tau=float(np.float32(0.07)), tau_img=f64(t_img),
                     tau_txt=f64(t_txt), tau_grad_scale=g.scale, u_glob_img=f64(ug1), u_glob_txt=f64(ug2),
                     tau_glob_img=f64(tg1), tau_glob_txt=f64(tg2))
    got = g.outputs()
    compare(got, want, version, tol, "gathered %s %s v%d" % (dtype, (B, b, off, d), version))
    check_state(g, u0i, u0t, idx, u_img, u_txt, tol)
    # the remote anchors' part is a sizeable share of the gradient: a path that dropped it could not pass
    local_only = fcco_step(img.astype(np.float64), txt.astype(np.float64), off, b, idx, u0i.astype(np.float64),
                           u0t.astype(np.float64), version=version, gamma=0.6, eps=g.eps, rho=g.rho,
                           tau=float(np.float32(0.07)), tau_img=f64(t_img), tau_txt=f64(t_txt), tau_grad_scale=g.scale)
    for k in ("d_img", "d_txt"):
        assert rel_l2(local_only[k], want[k]) > 20 * rel_l2(got[k], want[k])


@pytest.mark.parametrize("version", [V0, V1, V2, V3])
def test_f32_gathered_state(version):
    run_gathered(37, 11, 13, 19, version, "f32", TOL_F32, N=200, ld_pad=5)


@pytest.mark.parametrize("B,b,off,d", [(700, 300, 133, 72), (1000, 64, 936, 136), (768, 256, 256, 128),
                                       (1024, 300, 512, 256), (1536, 512, 512, 192), (1024, 300, 724, 256),
                                       (1024, 320, 704, 128)])
@pytest.mark.parametrize("version", [V0, V1, V2, V3])
def test_bf16_gathered_state(B, b, off, d, version):
    run_gathered(B, b, off, d, version, "bf16", TOL_BF16, ld_pad=8)


@pytest.mark.parametrize("B,b,off,d", [
    # one contrast tile of a pair, a second one that is short, columns wrapping inside a tile and inside a stage
    (100, 9, 91, 64), (300, 130, 57, 72), (257, 65, 3, 136), (1000, 64, 936, 520),
    # several splits; three groups of 256 local anchors; two rounds of output tiles, hence the state phase on its own
    (2048, 256, 768, 512), (5120, 640, 3200, 512), (1000, 520, 300, 1024)])
@pytest.mark.parametrize("version", [V0, V1, V2, V3])
def test_bf16_gathered_state_on_small_tiles(B, b, off, d, version):
    plan = fc.fastclip_describe(fc.make_config(version=version, emb_dtype=fc.BF16, B=B, b=b, off=off, d=d, N=5000, gamma=0.6,
                                               eps=1e-6, rho=6.5, ld_img=d + 8, ld_txt=d, flags=fc.GATHERED_STATE))
    assert plan["tile"] == 128 and plan["fused_state"] == (d < 1024) and (plan["nsplit"] > 1) == (B == 2048)
    run_gathered(B, b, off, d, version, "bf16", TOL_BF16, ld_pad=8, tiles=None)


@pytest.mark.parametrize("B,b,off,d,inside", [
    # state phase in the contraction, of one group of 256 local anchors and of three; on its own
    (300, 130, 57, 72, 1), (1000, 600, 200, 72, 1), (1000, 520, 300, 1024, 0)])
@pytest.mark.parametrize("version", [V2, V3])
def test_gathered_state_on_small_tiles_with_temperature_update(B, b, off, d, inside, version):
    """fastclip_step_update_tau with gathered state is fastclip_step followed by fastclip_temperature_update: the same bits
    in every output and in the state (one set of kernels), the temperatures and moments to a few units in the last place
    (the same arithmetic in another kernel, whose multiply-adds may be contracted differently)."""
    N = 3000
    rng = np.random.default_rng(B + version)
    img, txt = make_embeddings(B + 31, B, d, 0.5, "bf16")
    idx = draw_indices(B + 32, b, N)
    u0i, u0t = (rng.uniform(0.05, 2.0, N).astype(np.float32) for _ in range(2))
    t_img, t_txt = (rng.uniform(0.05, 0.1, N).astype(np.float32) for _ in range(2))
    ug1, ug2, tg1, tg2 = gathered_inputs(rng, B, version)
    upd = fc.make_tau_update(optimizer=ADAMW, step=3, lr=2e-3, beta1=0.9, beta2=0.98, eps=1e-6, tau_min=0.01)
    runs = []
    for fused in (True, False):
        g = GpuStep(B=B, b=b, off=off, d=d, N=N, dtype="bf16", version=version, eps=1e-6, rho=6.5, tau=0.07, u_img0=u0i,
                    u_txt0=u0t, tau_img0=t_img, tau_txt0=t_txt, gathered=dict(u_img=ug1, u_txt=ug2, tau_img=tg1, tau_txt=tg2),
                    tiles=None)
        plan = fc.fastclip_describe(g.config(0.6))
        assert plan["tile"] == 128 and plan["fused_state"] == inside
        g.set_inputs(img, txt, idx)
        z = lambda n: torch.full((n,), 0.01, dtype=torch.float32, device=DEV)
        moments = {k: z(N) for k in ("m_img", "v_img", "m_txt", "v_txt")} if version == V2 else dict(m=z(1), v=z(1))
        tau = dict(tau_img=g.tau_img, tau_txt=g.tau_txt) if version == V2 else dict(tau=g.tau)
        state = fc.make_tau_state(**tau, **moments)
        if fused:
            g.step_update_tau(0.6, upd, state)
        else:
            g.step(0.6)
            fc.fastclip_temperature_update(version, upd, state, g.idx, b, N, g.d_tau, g.d_tau_img, g.d_tau_txt)
            torch.cuda.synchronize()
        runs.append((g, dict(tau, **moments)))
    (g, s), (h, t) = runs
    for k in ("d_img", "d_txt", "loss", "d_tau", "d_tau_img", "d_tau_txt", "g_img", "g_txt", "u_new_img", "u_new_txt", "u_img", "u_txt"):
        assert torch.equal(getattr(g, k).view(torch.int32), getattr(h, k).view(torch.int32)), k
    for k in s:
        assert float((s[k] - t[k]).abs().max()) <= 8 * 2.0 ** -23 * float(t[k].abs().max()), k
    moved = s["tau_img"] if version == V2 else s["tau"]
    start = torch.from_numpy(t_img).to(DEV) if version == V2 else torch.full_like(moved, 0.07)
    assert int((moved != start).sum()) == (b if version == V2 else 1)


@pytest.mark.parametrize("b,d,ld,at", [(3, 4, 4, 0), (5, 1020, 1024, 0), (6, 516, 516, 4), (7, 512, 512, 1), (9, 1028, 1028, 0)])
def test_normalize_rows_alignment(b, d, ld, at):
    """Rows of whole aligned groups of four are held in registers; an odd start, a stride or width that is none, or a wider row
    takes the element-wise kernel: the same rows to the last bit of the rounding, whichever it is."""
    rng = np.random.default_rng(b * d)
    flat = np.full(at + b * ld + 8, np.nan, np.float32)
    raw = raw_rows(rng, b, d, "f32")
    for r in range(b):
        flat[at + r * ld: at + r * ld + d] = raw[r]
    t_raw = torch.from_numpy(flat).to(DEV)
    t_unit, t_norm = torch.full((b, ld), 7.5, device=DEV), torch.empty(b, device=DEV)
    fc.fastclip_normalize_rows(t_raw.data_ptr() + 4 * at, fc.F32, ld, b, d, t_unit, fc.F32, ld, t_norm)
    torch.cuda.synchronize()
    want, norm = normalize_rows(raw.astype(np.float64))
    assert rel_each(t_norm.cpu().numpy().astype(np.float64), norm) <= 2e-7
    # one rounding of 1 / |e| and one of the product: 2^-24 each
    assert np.all(np.abs(t_unit[:, :d].cpu().numpy().astype(np.float64) - want) <= (2.0 ** -23 + 3e-7) * np.abs(want))
    assert (t_unit[:, d:] == 7.5).all()


@pytest.mark.parametrize("B,b,off,d", [
    (200, 90, 100, 72),                           # six stages on the loop that forms the operand from both strips
    (256, 128, 0, 200), (288, 100, 150, 256),     # eight; nine, an odd run; output tiles of either width
    (520, 300, 217, 520), (700, 257, 443, 264), (1100, 513, 300, 768),      # several splits, odd ones, ragged rows and columns
    (2304, 300, 77, 392)])
def test_bf16_gathered_state_large_tiles_edges(B, b, off, d):
    """Contraction of the large tiles with gathered state at the depths and widths where its loop begins and ends."""
    run_gathered(B, b, off, d, V2 if d % 3 else V3, "bf16", TOL_BF16, ld_pad=8)


@pytest.mark.parametrize("stages", [1, 2, 3, 4, 5, 7, 11])
@pytest.mark.parametrize("d", [192, 256])
def test_bf16_gathered_state_large_tiles_runs_of_stages(stages, d):
    """... and where the whole stages of a split are few or an odd number; a row behind them is left to the guarded loop."""
    run_gathered(32 * stages + 1, 20, 9, d, V2 if stages % 2 else V3, "bf16", TOL_BF16, ld_pad=8)


def test_gathered_state_with_whole_batch_is_the_plain_step():
    """b == B: no remote anchors; the flag changes nothing and the gathered arrays are not read."""
    B, d, N = 520, 64, 5000
    img, txt = make_embeddings(11, B, d, 0.5, "bf16")
    idx = draw_indices(12, B, N)
    res = []
    for gathered in (None, dict(u_img=np.full(B, np.nan), u_txt=np.full(B, np.nan))):
        g = GpuStep(B=B, b=B, off=0, d=d, N=N, dtype="bf16", version=V3, eps=1e-14, rho=6.5, gathered=gathered)
        g.set_inputs(img, txt, idx)
        g.step(0.7)
        res.append((g.d_img.cpu(), g.d_txt.cpu(), g.u_img.cpu(), g.loss.cpu(), g.d_tau.cpu()))
    for x, y in zip(*res):
        assert torch.equal(x, y)


# ------------------------------------------------------------------------------- seeded random shapes
def random_case(rs, dtype):
    """A valid shape: sizes around the 256-tile edges, tiny ones, whole batches, local shares of every offset."""
    if dtype == "f32":
        B = int(rs.integers(2, 160))
        d = int(rs.integers(1, 70))
    else:
        kind = rs.integers(0, 6)
        B = int(rs.choice([255, 256, 257, 511, 512, 513, 767, 768, 769, 1023, 1024, 1025, 2047, 2048, 2049])) if kind == 0 \
            else int(rs.integers(2, 300)) if kind == 1 else int(rs.integers(300, 2500))
        d = int(rs.choice([8, 16, 24, 40, 64, 72, 96, 128, 136, 192, 200, 256, 264, 320]))
    mode = rs.integers(0, 5)
    b = B if mode == 0 else int(rs.integers(1, min(B, 40) + 1)) if mode == 1 else \
        int(min(B, 32 * rs.integers(1, 40))) if mode == 2 else int(rs.integers(1, B + 1))
    off = 0 if b == B else int(rs.choice([0, B - b, int(rs.integers(0, B - b + 1))]))
    return B, b, off, d


@pytest.mark.parametrize("dtype,tol,cases", [("bf16", TOL_BF16, 60), ("f32", TOL_F32, 40)])
def test_random_shapes(dtype, tol, cases):
    """Seeded draws of shape, version, gathered state, record stride, gamma and row strides against the oracle."""
    rs = np.random.default_rng(20240701)
    for case in range(cases):
        B, b, off, d = random_case(rs, dtype)
        version = int(rs.choice([V0, V1, V2, V3]))
        gathered = bool(rs.integers(0, 3) == 0) and b < B
        stride = int(rs.choice([1, 1, 4, 8]))
        gamma = float(rs.choice([0.6, 1.0, 0.25]))
        N = int(rs.integers(b, 4 * b + 100))
        pad = int(rs.choice([0, 8, 24]))
        normed = bool(rs.integers(0, 3) == 0)       # gradients with respect to rows that were normalised outside
        tiles = (256, None, 128)[case % 3]          # bf16: large tiles, the library's choice, small tiles where they apply
        print("[random %s %d] B=%d b=%d off=%d d=%d v%d gathered=%d stride=%d gamma=%.2f N=%d pad=%d normed=%d tiles=%s"
              % (dtype, case, B, b, off, d, version, gathered, stride, gamma, N, pad, normed, tiles), flush=True)
        rng = np.random.default_rng(case)
        img, txt = make_embeddings(case + 7, B, d, 0.5, dtype)
        idx = draw_indices(case + 3, b, N)
        u0i = np.where(rng.random(N) < 0.5, 0.0, rng.uniform(0.05, 2.0, N)).astype(np.float32)
        u0t = np.where(rng.random(N) < 0.5, 0.0, rng.uniform(0.05, 2.0, N)).astype(np.float32)
        t_img = rng.uniform(0.05, 0.1, N).astype(np.float32)
        t_txt = rng.uniform(0.05, 0.1, N).astype(np.float32)
        f64 = lambda a: None if a is None else a.astype(np.float64)
        gath, extra = None, {}
        if gathered:
            ug1, ug2, tg1, tg2 = gathered_inputs(rng, B, version)
            gath = dict(u_img=ug1, u_txt=ug2, tau_img=tg1, tau_txt=tg2)
            extra = dict(u_glob_img=f64(ug1), u_glob_txt=f64(ug2), tau_glob_img=f64(tg1), tau_glob_txt=f64(tg2))
        norms = None
        if normed:
            norms = (rng.uniform(0.3, 20.0, b).astype(np.float32), rng.uniform(0.3, 20.0, b).astype(np.float32))
            extra.update(norm_img=f64(norms[0]), norm_txt=f64(norms[1]))
        g = GpuStep(B=B, b=b, off=off, d=d, N=N, dtype=dtype, version=version, eps=1e-6, rho=6.5, tau=0.07,
                    tau_grad_scale=1.0 / N, ld_img=d + pad, ld_txt=d, u_img0=u0i, u_txt0=u0t, tau_img0=t_img,
                    tau_txt0=t_txt, gathered=gath, state_stride=stride, norms=norms, tiles=tiles)
        g.set_inputs(img, txt, idx)
        g.step(gamma)
        u_img, u_txt = u0i.astype(np.float64), u0t.astype(np.float64)
        want = fcco_step(img.astype(np.float64), txt.astype(np.float64), off, b, idx, u_img, u_txt, version=version,
                         gamma=gamma, eps=g.eps, rho=g.rho, tau=float(np.float32(0.07)), tau_img=f64(t_img),
                         tau_txt=f64(t_txt), tau_grad_scale=g.scale, **extra)
        compare(g.outputs(), want, version, tol, "random %s %d" % (dtype, case))
        check_state(g, u0i, u0t, idx, u_img, u_txt, tol)


# ------------------------------------------------------------------------------- temperature update (Alg. 1 line 12)
OPTIMIZERS = [(SGDM, dict(lr=1e-3, beta1=0.9, beta2=0.0)), (LAMB, dict(lr=1e-2, beta1=0.9, beta2=0.98, eps=1e-6)),
              (LION, dict(lr=1e-3, beta1=0.9, beta2=0.99)), (ADAMW, dict(lr=1e-2, beta1=0.9, beta2=0.999, eps=1e-8))]


@pytest.mark.parametrize("stride", [0, 6])
@pytest.mark.parametrize("opt,hp", OPTIMIZERS)
def test_temperature_update_alone(opt, hp, stride):
    """Proc. temperature_update from given gradients: per-sample (V2) and global (V3) temperatures; stride 6: the six
    per-sample arrays as the fields of one record per sample."""
    N, b, step = 5000, 300, 7
    rng = np.random.default_rng(100 + opt)
    idx = draw_indices(55, b, N)
    f32 = lambda lo, hi, n: rng.uniform(lo, hi, n).astype(np.float32)
    host = dict(tau_img=f32(0.02, 0.1, N), tau_txt=f32(0.02, 0.1, N), m_img=f32(-1, 1, N), m_txt=f32(-1, 1, N),
                v_img=f32(0.01, 2, N), v_txt=f32(0.01, 2, N))
    g_img, g_txt = f32(-3, 3, b), f32(-3, 3, b)
    extra = dict(tau_min=0.025, lr_drop_below=0.03, lr_drop_factor=1.0 / 3.0)
    if stride:
        rec = torch.from_numpy(np.stack([host[k] for k in host], axis=1)).to(DEV)
        dev = {k: rec[:, i] for i, k in enumerate(host)}
    else:
        dev = {k: torch.from_numpy(v).to(DEV) for k, v in host.items()}
    upd = fc.make_tau_update(optimizer=opt, step=step, state_stride=stride, **hp, **extra)
    fc.fastclip_temperature_update(V2, upd, fc.make_tau_state(**dev), torch.from_numpy(idx).to(DEV), b, N, None,
                                   torch.from_numpy(g_img).to(DEV), torch.from_numpy(g_txt).to(DEV))
    torch.cuda.synchronize()
    want = {k: v.astype(np.float64) for k, v in host.items()}
    temperature_update(V2, {"d_tau_img": g_img.astype(np.float64), "d_tau_txt": g_txt.astype(np.float64)},
                       optimizer=opt, step=step, idx=idx, **hp, **extra, **want)
    mask = np.ones(N, bool)
    mask[idx] = False
    for k in host:
        got = dev[k].cpu().numpy()
        assert np.array_equal(got[mask].view(np.uint32), host[k][mask].view(np.uint32)), k      # untouched entries
        if k.startswith("v_") and opt in (SGDM, LION):
            assert np.array_equal(got.view(np.uint32), host[k].view(np.uint32))                  # no second moment
            continue
        # temperatures: per element.  Moments: beta m + (1 - beta) G can cancel, so the fp32 rounding error is
        # bounded relative to the operands (max norm), not to each result
        if k.startswith("tau"):
            assert rel_each(got[idx], want[k][idx]) <= 1e-5, k
        else:
            assert rel_inf(got[idx], want[k][idx]) <= 1e-6, k
    assert (dev["tau_img"].cpu().numpy()[idx] >= np.float32(0.025)).all()
    # global temperature, below the threshold where the learning rate drops
    for tau0 in (0.07, 0.029):
        t, m, v, g = (torch.tensor([x], dtype=torch.float32, device=DEV) for x in (tau0, 0.3, 0.5, -1.7))
        fc.fastclip_temperature_update(V3, upd, fc.make_tau_state(tau=t, m=m, v=v), None, 0, 1, g, None, None)
        torch.cuda.synchronize()
        wt, wm, wv = temperature_update(V3, {"d_tau": float(np.float32(-1.7))}, optimizer=opt, step=step,
                                        tau=float(np.float32(tau0)), m=float(np.float32(0.3)),
                                        v=float(np.float32(0.5)), **hp, **extra)
        assert t.item() == pytest.approx(wt, rel=1e-5) and m.item() == pytest.approx(wm, rel=1e-5)
        if opt in (ADAMW, LAMB):
            assert v.item() == pytest.approx(wv, rel=1e-5)


@pytest.mark.parametrize("b", [1, 300])
def test_temperature_update_with_one_array_for_both_sides(b):
    """One temperature and one set of moments for both sides of a sample (V2): the image's step, then the text's from there."""
    N, step = 900, 4
    rng = np.random.default_rng(b)
    f32 = lambda lo, hi, n: rng.uniform(lo, hi, n).astype(np.float32)
    idx, g = draw_indices(56, b, N), [f32(-1, 1, b) for _ in range(2)]
    host = dict(tau=f32(0.05, 0.1, N), m=f32(-0.1, 0.1, N), v=f32(0.01, 0.05, N))
    dev = {k: torch.from_numpy(x.copy()).to(DEV) for k, x in host.items()}
    hp = {k: float(np.float32(x)) for k, x in dict(lr=2e-3, beta1=0.9, beta2=0.98, eps=1e-6).items()}
    upd = fc.make_tau_update(optimizer=ADAMW, step=step, **hp)
    both = lambda arrays: {k + side: x for k, x in arrays.items() for side in ("_img", "_txt")}
    t_idx, t_g = torch.from_numpy(idx).to(DEV), [torch.from_numpy(x).to(DEV) for x in g]
    fc.fastclip_temperature_update(V2, upd, fc.make_tau_state(**both(dev)), t_idx, b, N, None, t_g[0], t_g[1])
    torch.cuda.synchronize()
    want = {k: x.astype(np.float64) for k, x in host.items()}
    temperature_update(V2, dict(d_tau_img=g[0].astype(np.float64), d_tau_txt=g[1].astype(np.float64)), optimizer=ADAMW, step=step,
                       idx=idx, **hp, **both(want))
    for k in want:       # a dozen fp32 operations a step, each rounded once: 2^-24 of what they add up to, which is below 1
        assert np.max(np.abs(dev[k].cpu().numpy().astype(np.float64) - want[k])) <= 16 * 2.0 ** -24, k


@pytest.mark.parametrize("tiles", [256, None])   # the large-tile kernels; the library's choice (small tiles here)
@pytest.mark.parametrize("stride", [1, 8, "canonical 8", "canonical 16"])
@pytest.mark.parametrize("dtype,tol,shape", [("f32", TOL_F32, (64, 64, 0, 32)), ("bf16", TOL_BF16, (700, 300, 133, 72)),
                                             # enough anchors that the state phase is a kernel of its own on the large tiles
                                             # (on the small ones it rides along with four splits of the contraction)
                                             ("bf16", TOL_BF16, (2048, 1536, 256, 64))])
@pytest.mark.parametrize("version", [V2, V3, V0])
def test_step_with_temperature_update_three_iterations(dtype, tol, shape, version, stride, tiles):
    """fastclip_step_update_tau: step + temperature update per iteration, temperatures and moments carried on the
    device, against the oracle's step followed by Proc. temperature_update."""
    if dtype == "f32" and tiles is None:
        pytest.skip("the tile size concerns the bf16 path only")
    B, b, off, d = shape
    canonical = isinstance(stride, str)       # records {u_1, tau_1, m_1, v_1, u_2, tau_2, m_2, v_2}: 16-byte words per side
    stride = int(stride.split()[1]) if canonical else stride
    N = max(2000, 2 * b)
    rng = np.random.default_rng(9 + version)
    hp = dict(lr=2e-3, beta1=0.9, beta2=0.98, eps=1e-6)
    extra = dict(tau_min=0.01, lr_drop_below=0.03, lr_drop_factor=1.0 / 3.0)
    t_img0 = rng.uniform(0.05, 0.1, N).astype(np.float32)
    t_txt0 = rng.uniform(0.05, 0.1, N).astype(np.float32)
    g = GpuStep(B=B, b=b, off=off, d=d, N=N, dtype=dtype, version=version, eps=1e-6, rho=6.5, tau=0.07,
                tau_grad_scale=1.0, tau_img0=t_img0, tau_txt0=t_txt0, state_stride=stride, canonical_records=canonical, tiles=tiles)
    z = lambda n: torch.zeros(n, dtype=torch.float32, device=DEV)
    if version == V2 and canonical:
        for k in ("m_img", "v_img", "m_txt", "v_txt"):
            g.records[:, CANONICAL_FIELDS[k]] = 0.0
        st_dev = dict(tau_img=g.tau_img, tau_txt=g.tau_txt, **{k: g.records[:, CANONICAL_FIELDS[k]]
                                                                for k in ("m_img", "v_img", "m_txt", "v_txt")})
    elif version == V2 and stride > 1:     # the moments are fields 4..7 of the same records
        g.records[:, 4:8] = 0.0
        st_dev = dict(tau_img=g.tau_img, tau_txt=g.tau_txt, m_img=g.records[:, 4], v_img=g.records[:, 5],
                      m_txt=g.records[:, 6], v_txt=g.records[:, 7])
    elif version == V2:
        st_dev = dict(tau_img=g.tau_img, tau_txt=g.tau_txt, m_img=z(N), v_img=z(N), m_txt=z(N), v_txt=z(N))
    else:
        st_dev = dict(tau=g.tau, m=z(1), v=z(1))
    state = fc.make_tau_state(**st_dev)
    u_img, u_txt = np.zeros(N), np.zeros(N)
    w = dict(tau=float(np.float32(0.07)), m=0.0, v=0.0, tau_img=t_img0.astype(np.float64),
             tau_txt=t_txt0.astype(np.float64), m_img=np.zeros(N), v_img=np.zeros(N), m_txt=np.zeros(N),
             v_txt=np.zeros(N))
    for it in range(3):
        img, txt = make_embeddings(300 + it, B, d, 0.5, dtype)
        idx = draw_indices(400 + it, b, N)
        g.set_inputs(img, txt, idx)
        g.step_update_tau(0.7, fc.make_tau_update(optimizer=ADAMW, step=it + 1, state_stride=stride, **hp, **extra), state)
        want = fcco_step(img.astype(np.float64), txt.astype(np.float64), off, b, idx, u_img, u_txt, version=version,
                         gamma=0.7, eps=g.eps, rho=g.rho, tau=w["tau"], tau_img=w["tau_img"], tau_txt=w["tau_txt"],
                         tau_grad_scale=1.0)
        compare(g.outputs(), want, version, tol, "tau update %s v%d it %d" % (dtype, version, it))
        if version == V2:
            temperature_update(V2, want, optimizer=ADAMW, step=it + 1, idx=idx, tau_img=w["tau_img"],
                               tau_txt=w["tau_txt"], m_img=w["m_img"], v_img=w["v_img"], m_txt=w["m_txt"],
                               v_txt=w["v_txt"], **hp, **extra)
            for k in ("tau_img", "tau_txt", "m_img", "m_txt", "v_img", "v_txt"):
                got = st_dev[k].cpu().numpy().astype(np.float64)
                lim = 1e-4 if k.startswith("tau") else (tol if k.startswith("m") else 2 * tol)
                assert rel_inf(got, w[k]) <= lim, (k, it, rel_inf(got, w[k]))
                untouched = np.ones(N, bool)
                untouched[w["m_img"] != 0] = False
                assert np.array_equal(got[untouched], (t_img0 if k == "tau_img" else t_txt0 if k == "tau_txt"
                                                       else np.zeros(N, np.float32))[untouched].astype(np.float64)), k
        else:
            w["tau"], w["m"], w["v"] = temperature_update(version, want, optimizer=ADAMW, step=it + 1, tau=w["tau"],
                                                          m=w["m"], v=w["v"], **hp, **extra)
            assert st_dev["tau"].item() == pytest.approx(w["tau"], rel=1e-4)
            assert st_dev["m"].item() == pytest.approx(w["m"], rel=tol) and st_dev["v"].item() == pytest.approx(w["v"], rel=2 * tol)
    assert st_dev["tau_img" if version == V2 else "tau"].cpu().numpy().std() >= 0      # still finite
    assert np.isfinite(g.loss.item())
    if g.records is not None and stride > 8:
        assert (g.records[:, 8:] == RECORD_FILL).all()       # what lies behind the eight fields is never touched


@pytest.mark.parametrize("tiles", [256, None])   # the large-tile kernels; the library's choice (small tiles here)
# ------------------------------------------------------------------------------- cosine similarity, MBCL
@pytest.mark.parametrize("dtype,tol,shape", [("f32", TOL_F32, (37, 11, 13, 19)), ("f32", TOL_F32, (20, 9, 7, 70)),
                                             ("bf16", TOL_BF16, (700, 300, 133, 72)),
                                             ("bf16", TOL_BF16, (768, 512, 256, 128))])
@pytest.mark.parametrize("version", [V2, V3])
def test_gradients_through_normalisation(dtype, tol, shape, version, tiles):
    if dtype == "f32" and tiles is None:
        pytest.skip("the tile size concerns the bf16 path only")
    B, b, off, d = shape
    N = 3000
    rng = np.random.default_rng(B + version)
    img, txt = make_embeddings(B + 5, B, d, 0.5, dtype)
    idx = draw_indices(B + 6, b, N)
    n_img = rng.uniform(0.3, 20.0, b).astype(np.float32)          # what the rows measured before normalisation
    n_txt = rng.uniform(0.3, 20.0, b).astype(np.float32)
    t_img = rng.uniform(0.05, 0.1, N).astype(np.float32)
    t_txt = rng.uniform(0.05, 0.1, N).astype(np.float32)
    g = GpuStep(B=B, b=b, off=off, d=d, N=N, dtype=dtype, version=version, eps=1e-6, rho=6.5, tau=0.07,
                tau_grad_scale=1.0 / N, tau_img0=t_img, tau_txt0=t_txt, norms=(n_img, n_txt), tiles=tiles)
    g.set_inputs(img, txt, idx)
    g.step(0.6)
    want = fcco_step(img.astype(np.float64), txt.astype(np.float64), off, b, idx, np.zeros(N), np.zeros(N),
                     version=version, gamma=0.6, eps=g.eps, rho=g.rho, tau=float(np.float32(0.07)),
                     tau_img=t_img.astype(np.float64), tau_txt=t_txt.astype(np.float64), tau_grad_scale=g.scale,
                     norm_img=n_img.astype(np.float64), norm_txt=n_txt.astype(np.float64))
    compare(g.outputs(), want, version, tol, "normalised %s %s v%d" % (dtype, shape, version))


@pytest.mark.parametrize("dtype,tol,shape,pad", [
    # whole groups of four elements, a wavefront per row: one group, a lane's last word short of the row, the widest; wider rows and
    # a stride that is no multiple of four elements, a workgroup per row; a last workgroup of one anchor
    ("f32", TOL_F32, (40, 9, 7, 4), 0), ("f32", TOL_F32, (40, 21, 7, 260), 4), ("f32", TOL_F32, (40, 17, 3, 1024), 0),
    ("f32", TOL_F32, (40, 17, 3, 1028), 0), ("f32", TOL_F32, (40, 9, 7, 260), 3),
    ("bf16", TOL_BF16, (140, 65, 33, 8), 0), ("bf16", TOL_BF16, (140, 65, 33, 1024), 8), ("bf16", TOL_BF16, (140, 65, 33, 1032), 0)])
def test_gradients_through_normalisation_of_rows_of_any_width(dtype, tol, shape, pad):
    B, b, off, d = shape
    rng = np.random.default_rng(B + d)
    img, txt = make_embeddings(B + 5, B, d, 0.5, dtype)
    idx = draw_indices(B + 6, b, 3000)
    norms = [rng.uniform(0.3, 20.0, b).astype(np.float32) for _ in range(2)]
    g = GpuStep(B=B, b=b, off=off, d=d, N=3000, dtype=dtype, version=V3, eps=1e-6, rho=6.5, tau=0.07, norms=norms,
                ld_img=d + pad, ld_txt=d + pad)
    g.set_inputs(img, txt, idx)
    g.step(0.6)
    want = fcco_step(img.astype(np.float64), txt.astype(np.float64), off, b, idx, np.zeros(3000), np.zeros(3000), version=V3,
                     gamma=0.6, eps=g.eps, rho=g.rho, tau=float(np.float32(0.07)), tau_grad_scale=g.scale,
                     norm_img=norms[0].astype(np.float64), norm_txt=norms[1].astype(np.float64))
    compare(g.outputs(), want, V3, tol, "normalised %s %s" % (dtype, shape))


def raw_rows(rng, b, d, dtype):
    """Encoder outputs before normalisation: rows of very different lengths (values bf16-representable if dtype is bf16)."""
    raw = (rng.standard_normal((b, d)) * np.exp(rng.uniform(np.log(0.05), np.log(30.0), (b, 1)))).astype(np.float32)
    return round_to_bf16(raw) if dtype == "bf16" else raw


@pytest.mark.parametrize("raw_dtype,unit_dtype", [("f32", "f32"), ("f32", "bf16"), ("bf16", "bf16"), ("bf16", "f32")])
@pytest.mark.parametrize("b,d,pad", [(1, 1, 0), (5, 3, 2), (37, 19, 5), (300, 72, 8), (1024, 1024, 0), (130, 4104, 0)])
def test_normalize_rows(raw_dtype, unit_dtype, b, d, pad):
    """fastclip_normalize_rows against the oracle's e / |e| and |e|: norms to fp32 rounding, unit rows to the rounding
    of the storage type (half a unit in the last place of bf16 or fp32, plus the fp32 division)."""
    rng = np.random.default_rng(b + d)
    raw = raw_rows(rng, b, d, raw_dtype)
    if b > 2:
        raw[2] = 0.0                                                    # a row of zeros: zeros out, norm 0
    tdt = {"f32": torch.float32, "bf16": torch.bfloat16}
    t_raw = torch.full((b, d + pad), float("nan"), dtype=tdt[raw_dtype])
    t_raw[:, :d] = torch.from_numpy(raw).to(tdt[raw_dtype])
    t_raw = t_raw.to(DEV)
    t_unit = torch.full((b, d + 2 * pad), 7.5, dtype=tdt[unit_dtype], device=DEV)
    t_norm = torch.full((b,), float("nan"), dtype=torch.float32, device=DEV)
    code = {"f32": fc.F32, "bf16": fc.BF16}
    fc.fastclip_normalize_rows(t_raw, code[raw_dtype], d + pad, b, d, t_unit, code[unit_dtype], d + 2 * pad, t_norm)
    torch.cuda.synchronize()
    got_unit, got_norm = t_unit[:, :d].float().cpu().numpy().astype(np.float64), t_norm.cpu().numpy().astype(np.float64)
    keep = np.ones(b, bool)
    if b > 2:
        keep[2] = False
        assert got_norm[2] == 0.0 and (got_unit[2] == 0.0).all()
    want_unit, want_norm = normalize_rows(raw[keep].astype(np.float64))
    assert rel_each(got_norm[keep], want_norm) <= 2e-7
    half_ulp = 2.0 ** -8 if unit_dtype == "bf16" else 2.0 ** -24         # 8 and 24 significand bits
    assert np.all(np.abs(got_unit[keep] - want_unit) <= (half_ulp + 3e-7) * np.abs(want_unit) + 1e-30)
    if pad:
        assert (t_unit[:, d:].float() == 7.5).all()                     # nothing written beyond the row


@pytest.mark.parametrize("tiles", [256, None])   # the large-tile kernels; the library's choice (small tiles here)
@pytest.mark.parametrize("dtype,tol,shape", [("f32", TOL_F32, (37, 11, 13, 19)), ("f32", TOL_F32, (20, 9, 7, 70)),
                                             ("bf16", TOL_BF16, (700, 300, 133, 72)),
                                             ("bf16", TOL_BF16, (1024, 320, 704, 128))])
@pytest.mark.parametrize("version", [V2, V3])
def test_from_raw_encoder_rows_to_gradients_of_raw_rows(dtype, tol, shape, version, tiles):
    """The worker's whole boundary: its b raw image and text rows are normalised by the library into its slice of the
    global batch (cosine similarity, Sec. 3), the step runs on the unit rows with the norms it was handed, and d_img / d_txt
    are gradients with respect to the RAW rows.  The oracle normalises the same raw rows itself, rounds them to the
    storage type, and differentiates through the normalisation."""
    if dtype == "f32" and tiles is None:
        pytest.skip("the tile size concerns the bf16 path only")
    B, b, off, d = shape
    N = 3000
    rng = np.random.default_rng(B + 3 * version)
    img, txt = make_embeddings(B + 9, B, d, 0.5, dtype)                 # the other workers' rows, already unit rows
    raw_i, raw_t = raw_rows(rng, b, d, dtype), raw_rows(rng, b, d, dtype)
    raw_t = (raw_t + 2.0 * np.linalg.norm(raw_t, axis=1, keepdims=True) * raw_i / np.linalg.norm(raw_i, axis=1, keepdims=True)).astype(np.float32)
    if dtype == "bf16":
        raw_t = round_to_bf16(raw_t)
    idx = draw_indices(B + 10, b, N)
    t_img = rng.uniform(0.05, 0.1, N).astype(np.float32)
    t_txt = rng.uniform(0.05, 0.1, N).astype(np.float32)
    g = GpuStep(B=B, b=b, off=off, d=d, N=N, dtype=dtype, version=version, eps=1e-6, rho=6.5, tau=0.07,
                tau_grad_scale=1.0 / N, tau_img0=t_img, tau_txt0=t_txt,
                norms=(np.full(b, np.nan, np.float32), np.full(b, np.nan, np.float32)), tiles=tiles)
    g.set_inputs(img, txt, idx)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    code = fc.BF16 if dtype == "bf16" else fc.F32
    esz = 2 if dtype == "bf16" else 4
    for raw, glob, norm in ((raw_i, g.img, g.norm_img), (raw_t, g.txt, g.norm_txt)):
        t_raw = torch.from_numpy(raw).to(tdt).to(DEV)
        fc.fastclip_normalize_rows(t_raw, code, d, b, d, glob.data_ptr() + off * glob.stride(0) * esz, code, glob.stride(0), norm)
    g.step(0.6)
    # oracle side: its own normalisation of the same raw rows, rounded to the storage type like every other input
    img64, txt64 = img.astype(np.float64), txt.astype(np.float64)
    ui, ni = normalize_rows(raw_i.astype(np.float64))
    ut, nt = normalize_rows(raw_t.astype(np.float64))
    store = (lambda a: round_to_bf16(a.astype(np.float32)).astype(np.float64)) if dtype == "bf16" else \
        (lambda a: a.astype(np.float32).astype(np.float64))
    img64[off:off + b], txt64[off:off + b] = store(ui), store(ut)
    want = fcco_step(img64, txt64, off, b, idx, np.zeros(N), np.zeros(N), version=version, gamma=0.6, eps=g.eps, rho=g.rho,
                     tau=float(np.float32(0.07)), tau_img=t_img.astype(np.float64), tau_txt=t_txt.astype(np.float64),
                     tau_grad_scale=g.scale, norm_img=ni, norm_txt=nt)
    compare(g.outputs(), want, version, tol, "raw rows %s %s v%d" % (dtype, shape, version))


@pytest.mark.parametrize("dtype,tol,B,d", [("f32", TOL_F32, 64, 32), ("bf16", TOL_BF16, 520, 64),
                                          ("bf16", TOL_BF16, 512, 128)])
def test_mini_batch_contrastive_loss_is_a_special_case(dtype, tol, B, d):
    """The OpenCLIP-style mini-batch contrastive loss needs no code of its own: with zero state (u = g), V1 and
    eps = 1/M the step's gradient is that of tau (CE_rows(S/tau) + CE_cols(S/tau)) (softmax cross-entropy with the
    pairs on the diagonal), here taken from torch's log_softmax and autograd in fp64 on the CPU."""
    tau = float(np.float32(0.07))
    img, txt = make_embeddings(B + 31, B, d, 0.5, dtype)
    g = GpuStep(B=B, b=B, off=0, d=d, N=B, dtype=dtype, version=V1, eps=1.0 / (B - 1), tau=0.07)
    g.set_inputs(img, txt, np.arange(B))
    g.step(0.3)                                                # zero state: the first visit stores g whatever gamma is
    I = torch.tensor(img.astype(np.float64), requires_grad=True)
    T = torch.tensor(txt.astype(np.float64), requires_grad=True)
    S = I @ T.T / tau
    diag = torch.arange(B)
    ce = -(torch.log_softmax(S, dim=1)[diag, diag] + torch.log_softmax(S, dim=0)[diag, diag]).mean()
    (tau * ce).backward()
    assert rel_inf(g.d_img.cpu().numpy(), I.grad.numpy()) <= tol and rel_l2(g.d_img.cpu().numpy(), I.grad.numpy()) <= tol
    assert rel_inf(g.d_txt.cpu().numpy(), T.grad.numpy()) <= tol and rel_l2(g.d_txt.cpu().numpy(), T.grad.numpy()) <= tol
    # loss: tau/B sum [log(eps + g1) + log(eps + g2)] = tau (CE - 2 log M)
    assert g.loss.item() == pytest.approx(tau * (ce.item() - 2.0 * np.log(B - 1)), rel=tol, abs=tol * tau)


# ------------------------------------------------------------------------------- state kept as records
@pytest.mark.parametrize("dtype,shape", [("f32", (64, 64, 0, 32)), ("bf16", (700, 300, 133, 72))])
@pytest.mark.parametrize("version", [V2, V3])
def test_record_state_layout_is_the_dense_step(dtype, shape, version):
    """state_stride = 6: u_1, u_2, tau_1, tau_2 as fields of one record per sample.  Only addresses change, so every
    output and every state entry must equal the dense run bit for bit, and the other fields stay untouched."""
    B, b, off, d = shape
    N = 3000
    rng = np.random.default_rng(31 + version)
    img, txt = make_embeddings(17, B, d, 0.5, dtype)
    idx = draw_indices(18, b, N)
    u0i = np.where(rng.random(N) < 0.5, 0.0, rng.uniform(0.05, 2.0, N)).astype(np.float32)
    u0t = np.where(rng.random(N) < 0.5, 0.0, rng.uniform(0.05, 2.0, N)).astype(np.float32)
    t_img, t_txt = rng.uniform(0.05, 0.1, N).astype(np.float32), rng.uniform(0.05, 0.1, N).astype(np.float32)
    runs = []
    for stride in (1, 6):
        g = GpuStep(B=B, b=b, off=off, d=d, N=N, dtype=dtype, version=version, eps=1e-6, rho=6.5, tau=0.07,
                    tau_grad_scale=1.0 / N, u_img0=u0i, u_txt0=u0t, tau_img0=t_img, tau_txt0=t_txt, state_stride=stride)
        g.set_inputs(img, txt, idx)
        g.step(0.6)
        runs.append(g)
    dense, rec = runs
    for k, v in dense.outputs().items():
        assert np.array_equal(np.asarray(v), np.asarray(rec.outputs()[k]), equal_nan=True), k
    assert torch.equal(dense.u_img, rec.u_img.contiguous()) and torch.equal(dense.u_txt, rec.u_txt.contiguous())
    first_free = 4 if version == V2 else 2
    assert (rec.records[:, first_free:] == RECORD_FILL).all()
    if version == V2:
        assert torch.equal(rec.tau_img.contiguous(), dense.tau_img) and torch.equal(rec.tau_txt.contiguous(), dense.tau_txt)


# ------------------------------------------------------------------------------- full-size workloads
# What the MFMA path has been measured to reach on the full-size workloads is 6e-6 .. 6e-5 (the bf16 rounding of the
# stored exponentials averages out over thousands of terms); the guard sits a little above that, a factor ten below
# the contractual 2e-2, so that a term that is dropped or mis-scaled by a few per cent cannot hide under the contract.
TOL_BF16_MEASURED = 2e-3


def run_workload(name, steps_checked, n_steps, gathered=False, own_trajectory=False, needs_contrast_side=False,
                 tiles=None):
    """tiles: None = the tile size the library chooses, which is what bench.py times; 256 = the large-tile kernels.
    own_trajectory: the oracle carries its own state arrays through all steps (else it is handed the GPU's state of
    the batch's samples before each checked step).  needs_contrast_side: also check that the result could not pass
    without the local anchors' part of Eqs. 3 / 5 / 7."""
    w = WORKLOADS[name]
    B, b, off, d, N, version = w["B"], w["b"], w["off"], w["d"], w["N"], w["version"]
    gath, gath64 = None, {}
    if gathered:
        ug1, ug2, tg1, tg2 = gathered_inputs(np.random.default_rng(step_seed(name, 77)), B, version)
        gath = dict(u_img=ug1, u_txt=ug2, tau_img=tg1, tau_txt=tg2)
        gath64 = dict(u_glob_img=ug1.astype(np.float64), u_glob_txt=ug2.astype(np.float64),
                      tau_glob_img=None if tg1 is None else tg1.astype(np.float64),
                      tau_glob_txt=None if tg2 is None else tg2.astype(np.float64))
    g = GpuStep(B=B, b=b, off=off, d=d, N=N, dtype=w["dtype"], version=version, eps=w["eps"], rho=w["rho"],
                tau=w["tau"], tau_grad_scale=1.0 / N, gathered=gath, tiles=tiles)
    tau32 = float(np.float32(w["tau"]))
    own_u_img, own_u_txt = (np.zeros(N), np.zeros(N)) if own_trajectory else (None, None)
    for step in range(n_steps):
        gamma = w["gamma"] if not isinstance(w["gamma"], tuple) else gamma_cosine(step, 1, w["gamma"][1], w["gamma"][2])
        seed = step_seed(name, step)
        img, txt = make_embeddings(seed, B, d, w["noise"], w["dtype"])      # a fresh batch every step
        idx = draw_indices(seed + 500, b, N)
        g.set_inputs(img, txt, idx)
        if step not in steps_checked and not own_trajectory:
            g.step(gamma)
            continue
        idx_t = torch.from_numpy(idx).to(DEV)
        if own_trajectory:
            # the oracle's own state (never sees a value from the GPU), on a compact copy indexed 0..b-1
            u_img_c, u_txt_c = own_u_img[idx], own_u_txt[idx]
        else:
            # the oracle sees the state as the GPU holds it before the step
            u_img_c = g.u_img[idx_t].cpu().numpy().astype(np.float64)
            u_txt_c = g.u_txt[idx_t].cpu().numpy().astype(np.float64)
        checked = step in steps_checked
        if checked:
            keep_img, keep_txt = g.u_img.clone(), g.u_txt.clone()
            print("[%s] step %d gamma %.4f" % (name, step, gamma), flush=True)
        g.step(gamma)
        tau_c = np.full(b, tau32)
        f64 = lambda a: a.astype(np.float64)
        u_before = (u_img_c.copy(), u_txt_c.copy())
        want = fcco_step(f64(img), f64(txt), off, b, np.arange(b), u_img_c, u_txt_c, version=version, gamma=gamma,
                         eps=w["eps"], rho=w["rho"], tau=tau32, tau_img=tau_c, tau_txt=tau_c, tau_grad_scale=1.0 / N,
                         **gath64)
        if own_trajectory:
            own_u_img[idx], own_u_txt[idx] = u_img_c, u_txt_c
        if not checked:
            continue
        got = g.outputs()
        compare(got, want, version, TOL_BF16, "%s%s step %d" % (name, " gathered" if gathered else "", step),
                tol_measured=TOL_BF16_MEASURED)
        if needs_contrast_side:
            without = fcco_step(f64(img), f64(txt), off, b, np.arange(b), u_before[0], u_before[1], version=version,
                                gamma=gamma, eps=w["eps"], rho=w["rho"], tau=tau32, tau_img=tau_c, tau_txt=tau_c,
                                tau_grad_scale=1.0 / N, contrast_side=False)
            for k in ("d_img", "d_txt"):
                missing, err = rel_l2(without[k], want[k]), rel_l2(got[k], want[k])
                print("[%s] %s: the local contrast-side term is %.2e of the gradient, error %.2e" % (name, k, missing, err),
                      flush=True)
                assert missing > 20 * err
        # state: scattered values are the reported ones, everything else is bit-identical
        assert torch.equal(g.u_img[idx_t], g.u_new_img) and torch.equal(g.u_txt[idx_t], g.u_new_txt)
        keep_img[idx_t] = g.u_new_img
        keep_txt[idx_t] = g.u_new_txt
        assert torch.equal(keep_img.view(torch.int32), g.u_img.view(torch.int32))
        assert torch.equal(keep_txt.view(torch.int32), g.u_txt.view(torch.int32))
        assert rel_each(g.u_new_img.cpu().numpy(), u_img_c) <= TOL_BF16
        del keep_img, keep_txt
    if own_trajectory:      # the whole state after all steps, every entry: visited ones within tolerance, the rest zero
        for dev_u, own in ((g.u_img, own_u_img), (g.u_txt, own_u_txt)):
            got_u = dev_u.cpu().numpy().astype(np.float64)
            seen = own != 0
            assert np.array_equal(got_u != 0, seen)
            assert rel_each(got_u[seen], own[seen]) <= TOL_BF16_MEASURED
    return g


@pytest.mark.parametrize("tiles", [None, 256])
def test_cfg1_full_size(tiles):
    """100 steps with the cosine gamma schedule, a fresh batch every step, the state carried on the GPU and, on its
    own, by the oracle (which never sees a value of the GPU's); every output compared at the first, second, middle and
    last step, the whole state after the last."""
    run_workload("cfg1", {0, 1, 50, 99}, 100, own_trajectory=True, tiles=tiles)


@pytest.mark.parametrize("tiles", [None, 256])
def test_cfg2_full_size(tiles):
    run_workload("cfg2", {0, 2}, 3, needs_contrast_side=True, tiles=tiles)


def test_cfg3_full_size():
    run_workload("cfg3", {0, 1}, 2)


def test_cfg4_full_size():
    run_workload("cfg4", {0, 1}, 2, needs_contrast_side=True)


def test_cfg2_full_size_gathered_state():
    run_workload("cfg2", {0, 2}, 3, gathered=True)


def test_cfg4_full_size_gathered_state():
    run_workload("cfg4", {1}, 2, gathered=True)


# ------------------------------------------------------------------------------- auxiliary entry points
def test_check_indices_on_device():
    N = 1_000_000
    for b in (1, 64, 1000, 100_000):
        idx = draw_indices(b, b, N)
        ws = torch.empty(fc.fastclip_check_indices_workspace_bytes(b), dtype=torch.uint8, device=DEV)
        t = torch.from_numpy(idx).to(DEV)
        assert fc.fastclip_check_indices(t, b, N, ws) == fc.OK
        if b > 1:
            dup = idx.copy()
            dup[b // 2] = dup[0]
            assert fc.fastclip_check_indices(torch.from_numpy(dup).to(DEV), b, N, ws) == fc.ERR_INDEX
        for bad in (-1, N):
            oob = idx.copy()
            oob[-1] = bad
            assert fc.fastclip_check_indices(torch.from_numpy(oob).to(DEV), b, N, ws) == fc.ERR_INDEX


def test_state_update_alone_on_records():
    """fastclip_state_update_strided on records {u_1, u_2, free}: bit for bit the dense call."""
    N, n = 200_000, 50_000
    rng = np.random.default_rng(5)
    idx = torch.from_numpy(draw_indices(6, n, N)).to(DEV)
    u0 = torch.from_numpy(np.where(rng.random((N, 2)) < 0.5, 0.0, rng.uniform(0.05, 2.0, (N, 2))).astype(np.float32)).to(DEV)
    s1 = torch.from_numpy(rng.uniform(1.0, 900.0, n).astype(np.float32)).to(DEV)
    s2 = torch.from_numpy(rng.uniform(1.0, 900.0, n).astype(np.float32)).to(DEV)
    ui, ut = u0[:, 0].contiguous(), u0[:, 1].contiguous()
    o = [torch.empty(n, device=DEV) for _ in range(4)]
    fc.fastclip_state_update(idx, n, N, 0.4, 1023.0, s1, s2, ui, ut, o[0], o[1])
    rec = torch.full((N, 3), RECORD_FILL, dtype=torch.float32, device=DEV)
    rec[:, :2] = u0
    fc.fastclip_state_update_strided(idx, n, N, 3, 0.4, 1023.0, s1, s2, rec[:, 0], rec[:, 1], o[2], o[3])
    torch.cuda.synchronize()
    assert torch.equal(o[0], o[2]) and torch.equal(o[1], o[3])
    assert torch.equal(rec[:, 0].contiguous(), ui) and torch.equal(rec[:, 1].contiguous(), ut)
    assert (rec[:, 2] == RECORD_FILL).all()
    assert fc.fastclip_state_update_strided(idx, n, N, 0, 0.4, 1023.0, s1, s2, ui, ut, o[0], o[1], check=False) == fc.ERR_SHAPE


STATE_LAYOUTS = ["dense", "records 8", "records 16", "fields in another order"]


@pytest.mark.parametrize("update", [False, True])
@pytest.mark.parametrize("dtype,tol", [("f32", TOL_F32), ("bf16", 1e-4)])
@pytest.mark.parametrize("version", [V0, V1, V2, V3])
def test_state_phase_alone(version, dtype, tol, update):
    """fastclip_state_phase (the step's state kernel given the sums over the contrasts) against the oracle's step on
    a small problem whose sums the oracle supplies; the dense arrays, canonical records of 8 and 16 floats (one 16-byte
    word per side) and records with the fields in another order must give the same bits.  bf16 here only selects the
    fp32 logarithms of the MFMA path: from identical sums that path agrees with the oracle to 1e-4, not 2e-2."""
    B, b, off, d, N = 300, 300, 0, 16, 1500
    n = b
    rng = np.random.default_rng(70 + version)
    img, txt = make_embeddings(71, B, d, 0.5, "f32")
    idx = draw_indices(72, n, N)
    u0i = np.where(rng.random(N) < 0.5, 0.0, rng.uniform(0.05, 2.0, N)).astype(np.float32)
    u0t = np.where(rng.random(N) < 0.5, 0.0, rng.uniform(0.05, 2.0, N)).astype(np.float32)
    t_img = rng.uniform(0.05, 0.1, N).astype(np.float32)
    t_txt = rng.uniform(0.05, 0.1, N).astype(np.float32)
    m0 = {k: rng.uniform(-1, 1, N).astype(np.float32) for k in ("m_img", "m_txt")}
    v0 = {k: rng.uniform(0.01, 2, N).astype(np.float32) for k in ("v_img", "v_txt")}
    tau32, gamma, eps, rho, scale = float(np.float32(0.07)), 0.6, 1e-6, 6.5, 0.25
    u_img, u_txt = u0i.astype(np.float64), u0t.astype(np.float64)
    want = fcco_step(img.astype(np.float64), txt.astype(np.float64), off, b, idx, u_img, u_txt, version=version,
                     gamma=gamma, eps=eps, rho=rho, tau=tau32, tau_img=t_img.astype(np.float64),
                     tau_txt=t_txt.astype(np.float64), tau_grad_scale=scale)
    M = B - 1
    sums = np.stack([M * want["g_img"], M * want["h_img"], M * want["g_txt"], M * want["h_txt"]]).astype(np.float32)
    hp = dict(optimizer=ADAMW, step=3, lr=2e-3, beta1=0.9, beta2=0.98, eps=1e-6)
    extra = dict(tau_min=0.01, lr_drop_below=0.06, lr_drop_factor=1.0 / 3.0)
    w = dict(tau=tau32, m=0.3, v=0.5, tau_img=t_img.astype(np.float64), tau_txt=t_txt.astype(np.float64),
             **{k: a.astype(np.float64) for k, a in {**m0, **v0}.items()})
    if update and version == V2:
        temperature_update(V2, want, idx=idx, **hp, **extra, **{k: w[k] for k in ("tau_img", "tau_txt", "m_img", "v_img", "m_txt", "v_txt")})
    elif update and version != V1:
        w["tau"], w["m"], w["v"] = temperature_update(version, want, tau=w["tau"], m=w["m"], v=w["v"], **hp, **extra)
    host = dict(u_img=u0i, u_txt=u0t, tau_img=t_img, tau_txt=t_txt, **m0, **v0)
    results = []
    for layout in STATE_LAYOUTS:
        f32 = dict(dtype=torch.float32, device=DEV)
        if layout == "dense":
            stride, fields = 1, {k: torch.from_numpy(a).to(DEV) for k, a in host.items()}
        else:
            stride = 16 if layout == "records 16" else 8
            cols = CANONICAL_FIELDS if layout != "fields in another order" else \
                dict(u_img=0, u_txt=1, tau_img=2, tau_txt=3, m_img=4, v_img=5, m_txt=6, v_txt=7)
            rec = torch.full((N, stride), RECORD_FILL, **f32)
            for k, a in host.items():
                rec[:, cols[k]] = torch.from_numpy(a).to(DEV)
            fields = {k: rec[:, cols[k]] for k in host}
        tau_t, m_t, v_t = (torch.tensor([x], **f32) for x in (0.07, 0.3, 0.5))
        out = {k: torch.full((n,), float("nan"), **f32) for k in ("d_tau_img", "d_tau_txt", "g_img", "g_txt", "u_new_img", "u_new_txt")}
        loss, d_tau = torch.full((1,), float("nan"), **f32), torch.full((1,), float("nan"), **f32)
        coef = torch.full((3, n), float("nan"), **f32)
        cfg = fc.make_config(version=version, emb_dtype=fc.BF16 if dtype == "bf16" else fc.F32, B=B, b=b, off=off, d=d, N=N,
                             gamma=gamma, eps=eps, rho=rho, tau_grad_scale=scale, state_stride=stride)
        bufs = fc.make_buffers(idx=torch.from_numpy(idx).to(DEV), u_img=fields["u_img"], u_txt=fields["u_txt"], tau=tau_t,
                               tau_img=fields["tau_img"], tau_txt=fields["tau_txt"], loss=loss, d_tau=d_tau, **out)
        upd = state = None
        if update:
            upd = fc.make_tau_update(state_stride=stride, **hp, **extra)
            state = fc.make_tau_state(tau=tau_t, m=m_t, v=v_t, **{k: fields[k] for k in ("tau_img", "tau_txt", "m_img", "v_img", "m_txt", "v_txt")})
        ws = torch.empty(fc.fastclip_state_phase_workspace_bytes(n), dtype=torch.uint8, device=DEV)
        fc.fastclip_state_phase(cfg, bufs, upd, state, torch.from_numpy(sums).to(DEV), coef, ws)
        torch.cuda.synchronize()
        got = {k: t.cpu().numpy().astype(np.float64) for k, t in out.items()}
        got.update(loss=float(loss.item()), d_tau=float(d_tau.item()), d_img=want["d_img"], d_txt=want["d_txt"])
        compare(got, want, version, tol, "state phase %s v%d %s update=%d" % (dtype, version, layout, update))
        # the coefficients of Eqs. 2-7 from the oracle's u^{t+1} (V0: divided by tau)
        kappa = (1.0 / t_img[idx].astype(np.float64) if version == V2 else 1.0 / tau32) if version == V0 else 1.0
        kappa2 = (1.0 / t_txt[idx].astype(np.float64) if version == V2 else 1.0 / tau32) if version == V0 else 1.0
        c = coef.cpu().numpy().astype(np.float64)
        assert rel_each(c[0], kappa / (b * M * (eps + want["u_new_img"]))) <= tol
        assert rel_each(c[1], kappa2 / (b * M * (eps + want["u_new_txt"]))) <= tol
        assert rel_each(c[2], c[0] * sums[0] + c[1] * sums[2]) <= 1e-6
        state_now = {k: t.contiguous().cpu().numpy() for k, t in fields.items()}
        mask = np.ones(N, bool)
        mask[idx] = False
        for k, a in host.items():
            assert np.array_equal(state_now[k][mask].view(np.uint32), a[mask].view(np.uint32)), (k, layout)   # untouched
        assert np.array_equal(state_now["u_img"][idx], out["u_new_img"].cpu().numpy())
        if update and version == V2:
            for k in ("tau_img", "tau_txt", "m_img", "v_img", "m_txt", "v_txt"):
                lim = 1e-4 if k.startswith("tau") else 10 * tol
                assert rel_inf(state_now[k][idx], w[k][idx]) <= lim, (k, layout)
        else:
            for k in ("tau_img", "tau_txt", "m_img", "v_img", "m_txt", "v_txt"):
                assert np.array_equal(state_now[k].view(np.uint32), host[k].view(np.uint32)), (k, layout)
        if update and version in (V0, V3):
            assert tau_t.item() == pytest.approx(w["tau"], rel=1e-4) and m_t.item() == pytest.approx(w["m"], rel=10 * tol)
        if layout != "dense":
            assert (rec[:, 8:] == RECORD_FILL).all()
        results.append((state_now, {k: t.cpu().numpy() for k, t in out.items()}, coef.cpu().numpy(), loss.item(), d_tau.item()))
    for other in results[1:]:                 # every layout: the same bits
        for k in host:
            assert np.array_equal(other[0][k].view(np.uint32), results[0][0][k].view(np.uint32)), k
        for k in other[1]:
            assert np.array_equal(other[1][k], results[0][1][k], equal_nan=True), k
        assert np.array_equal(other[2], results[0][2]) and np.array_equal([other[3], other[4]], [results[0][3], results[0][4]], equal_nan=True)


@pytest.mark.parametrize("n", [1, 1000, 1 << 18])
def test_state_update_alone(n):
    N = 3_000_000
    rng = np.random.default_rng(n)
    idx = draw_indices(n + 7, n, N)
    u0i = np.where(rng.random(N) < 0.5, 0.0, rng.uniform(0.05, 2.0, N)).astype(np.float32)
    u0t = np.where(rng.random(N) < 0.5, 0.0, rng.uniform(0.05, 2.0, N)).astype(np.float32)
    s1 = rng.uniform(1.0, 900.0, n).astype(np.float32)
    s2 = rng.uniform(1.0, 900.0, n).astype(np.float32)
    M, gamma = 1023.0, 0.4
    dev = lambda a: torch.from_numpy(a).to(DEV)
    ui, ut, o1, o2 = dev(u0i), dev(u0t), torch.empty(n, device=DEV), torch.empty(n, device=DEV)
    fc.fastclip_state_update(dev(idx), n, N, gamma, M, dev(s1), dev(s2), ui, ut, o1, o2)
    torch.cuda.synchronize()
    wi, wt = u0i.astype(np.float64), u0t.astype(np.float64)
    n1 = ema_update(wi, idx, s1.astype(np.float64) / M, gamma)
    n2 = ema_update(wt, idx, s2.astype(np.float64) / M, gamma)
    assert rel_each(o1.cpu().numpy(), n1) <= 1e-6 and rel_each(o2.cpu().numpy(), n2) <= 1e-6
    got_i, got_t = ui.cpu().numpy(), ut.cpu().numpy()
    assert np.array_equal(got_i[idx], o1.cpu().numpy()) and np.array_equal(got_t[idx], o2.cpu().numpy())
    mask = np.ones(N, bool)
    mask[idx] = False
    assert np.array_equal(got_i[mask].view(np.uint32), u0i[mask].view(np.uint32))
    assert np.array_equal(got_t[mask].view(np.uint32), u0t[mask].view(np.uint32))


@pytest.mark.parametrize("tiles", [256, None])   # the large-tile kernels; the library's choice (small tiles here)
@pytest.mark.parametrize("shape,version", [((768, 512, 256, 128), V2), ((700, 300, 133, 72), V3)])
def test_step_replayed_from_a_hip_graph_equals_the_eager_step(shape, version, tiles):
    """The step allocates nothing and records no memset, so a caller may capture it in a HIP graph: every replay, on
    new inputs copied into the captured buffers and with eager work in between, equals the eager step bit for bit
    (state carried from replay to replay on both sides)."""
    B, b, off, d = shape
    N = 4000
    mk = lambda: GpuStep(B=B, b=b, off=off, d=d, N=N, dtype="bf16", version=version, eps=1e-6, rho=6.5, tau=0.07,
                         tau_grad_scale=1.0 / N, tiles=tiles)
    eager, cap = mk(), mk()
    inputs = [(make_embeddings(70 + i, B, d, 0.5, "bf16"), draw_indices(80 + i, b, N)) for i in range(4)]
    (img, txt), idx = inputs[0]
    cap.set_inputs(img, txt, idx)               # the captured buffers; later inputs are copied into them
    cfg = cap.config(0.7)
    ws = torch.empty(fc.fastclip_workspace_bytes(cfg), dtype=torch.uint8, device=DEV)
    bufs = cap.buffers()
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        fc.fastclip_step(cfg, bufs, ws)
    for (img, txt), idx in inputs:
        eager.set_inputs(img, txt, idx)
        eager.step(0.7)
        fresh = mk()
        fresh.set_inputs(img, txt, idx)
        cap.img.copy_(fresh.img)
        cap.txt.copy_(fresh.txt)
        cap.idx.copy_(fresh.idx)
        graph.replay()
        torch.cuda.synchronize()
        for k in ("d_img", "d_txt", "loss", "u_new_img", "u_new_txt", "u_img", "u_txt", "d_tau", "d_tau_img"):
            x, y = getattr(eager, k), getattr(cap, k)
            assert torch.equal(x.view(torch.int32), y.view(torch.int32)), k


def test_step_timed_reports_phases_and_same_result():
    B, b, off, d, N = 700, 300, 133, 72, 5000
    img, txt = make_embeddings(3, B, d, 0.5, "bf16")
    idx = draw_indices(4, b, N)
    outs = []
    for timed in (False, True):
        g = GpuStep(B=B, b=b, off=off, d=d, N=N, dtype="bf16", version=V0, eps=1e-14)
        g.set_inputs(img, txt, idx)
        ms = g.step(0.7, timed=timed)
        outs.append((g.d_img.cpu(), g.u_img.cpu(), g.d_tau.cpu()))
    assert set(ms) == {"prep", "strips", "state", "local", "contract", "finalize"}
    assert all(v > 0 for k, v in ms.items() if k != "state") and ms["state"] >= 0     # few anchors: state runs inside "local"
    for x, y in zip(*outs):
        assert torch.equal(x, y)


def test_measurement_entries_run_and_leave_the_step_intact():
    """The measurement aids (MFMA ceiling, bare record read-modify-write, strip kernel variants) run, report sane figures,
    and a step after them still agrees with the step before them bit for bit."""
    B, b, off, d, N = 2048, 512, 512, 128, 20000
    img, txt = make_embeddings(5, B, d, 0.5, "bf16")
    idx = draw_indices(6, b, N)
    runs = []
    for measure in (False, True):
        g = GpuStep(B=B, b=b, off=off, d=d, N=N, dtype="bf16", version=V3, eps=1e-6, rho=6.5)
        g.set_inputs(img, txt, idx)
        if measure:
            cfg = g.config(0.7)
            ws = torch.empty(fc.fastclip_workspace_bytes(cfg) + fc.MEASURE_STRIPS_EXTRA_BYTES, dtype=torch.uint8, device=DEV)
            for abl in (0, 1, 2, 3, 4, 7):
                r = fc.fastclip_measure_strips(cfg, g.buffers(), ws, abl, reps=2)
                assert r["ms"] > 0 and r["workgroups"] == 2 * 2 * 8 and 0.5 < r["ghz"] < 3.0
                assert r["cycles_older_wave"] > 64 * 32 * r["stages_per_workgroup"] * 0.4       # the MFMAs were not optimised away
            mc = fc.fastclip_measure_mfma_ceiling(64, 256, torch.empty(64 * 128 + 2048, dtype=torch.uint8, device=DEV))
            assert 100 < mc["tflops"] < 2600 and 30 < mc["cycles_per_mfma"] < 80
            rec = torch.zeros(N, 8, dtype=torch.float32, device=DEV)
            fc.fastclip_measure_record_rmw(g.idx, b, N, rec, 8)
            torch.cuda.synchronize()
            touched = (rec != 0).any(dim=1)
            assert int(touched.sum()) == b and bool(touched[g.idx].all()) and bool((rec[g.idx] == 0.25).all())
        g.step(0.7)
        runs.append((g.d_img.cpu(), g.d_txt.cpu(), g.u_img.cpu(), g.loss.cpu(), g.d_tau.cpu()))
    for x, y in zip(*runs):
        assert torch.equal(x, y)
