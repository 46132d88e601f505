"""The kernels' own sources, compiled for the host against a stand-in for the HIP runtime and the gfx950 builtins
(tests/emu), run one small step per code path under AddressSanitizer and are compared with the oracle.

What this can show: an access outside a buffer (every buffer is an exact-size allocation, the matrices end with the
last row's d elements), a barrier that not every thread reaches (the run would hang: bounded by a time-out), wrong
indexing (the outputs would disagree with the oracle).  What it cannot: timing, the asynchrony of direct-to-LDS loads
(they copy at once here), anything the GPU compiler does.  It is also the only place where the opt-in fine-tile path
runs as long as it is kept off the GPU."""
from __future__ import annotations

import os
import re
import subprocess
import sys

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, os.path.join(ROOT, "tests", "emu"))
import build_emu  # noqa: E402

from oracle import ADAMW, LION, SGDM, V0, V1, V2, V3, ema_update, fcco_step, normalize_rows, temperature_update  # noqa: E402
from paper_2407_01445_amd import binding as fc  # noqa: E402
from paper_2407_01445_amd.workloads import draw_indices, make_embeddings  # noqa: E402

pytestmark = pytest.mark.skipif(build_emu.host_compiler() is None, reason="no host clang++ to build the emulation with")


# FASTCLIP_EMU_SANITIZER=thread (missing barriers show as data races on the LDS arrays) or =memory (with the workspace
# and the outputs left uninitialised: a value nobody wrote that reaches a branch, an address or an output) instead of
# the default AddressSanitizer; all three are clean on every case below.
SANITIZER = os.environ.get("FASTCLIP_EMU_SANITIZER", "address")


@pytest.fixture(scope="module")
def emu_step():
    return build_emu.build("-fsanitize=" + SANITIZER)


def bf16_bits(x32):
    return (np.ascontiguousarray(x32, np.float32).view(np.uint32) >> 16).astype(np.uint16)


def run_case(exe, tmp_path, *, B, b, off, d, version, dtype="bf16", flags=0, ld_img=None, ld_txt=None, N=900, tau=0.07,
             eps=1e-6, rho=6.5, gamma=0.6, seed=1, gathered=False):
    ld_img, ld_txt = ld_img or d, ld_txt or d
    rng = np.random.default_rng(seed)
    img, txt = make_embeddings(seed + 41, B, d, 0.5, dtype)
    idx = draw_indices(seed + 42, b, N)
    u0i = np.where(rng.random(N) < 0.5, 0.0, rng.uniform(0.05, 2.0, N)).astype(np.float32)
    u0t = np.where(rng.random(N) < 0.5, 0.0, rng.uniform(0.05, 2.0, N)).astype(np.float32)
    t_img = rng.uniform(0.05, 0.1, N).astype(np.float32)
    t_txt = rng.uniform(0.05, 0.1, N).astype(np.float32)
    glob = None
    if gathered:       # u^{t+1} and temperatures of every global row as other workers would have sent them
        glob = dict(u_img=rng.uniform(0.05, 2.0, B).astype(np.float32), u_txt=rng.uniform(0.05, 2.0, B).astype(np.float32),
                    tau_img=rng.uniform(0.05, 0.1, B).astype(np.float32), tau_txt=rng.uniform(0.05, 0.1, B).astype(np.float32))
        flags |= fc.GATHERED_STATE

    def matrix(x, ld):            # row stride ld, NaN in the padding, no padding behind the last row
        full = np.full((B, ld), np.nan, np.float32)
        full[:, :d] = x
        flat = full.reshape(-1)[: (B - 1) * ld + d]
        return bf16_bits(flat) if dtype == "bf16" else flat

    fin, fout = str(tmp_path / "case.in"), str(tmp_path / "case.out")
    with open(fin, "wb") as f:
        np.array([version, fc.BF16 if dtype == "bf16" else fc.F32, flags, B, b, off, d, ld_img, ld_txt, N, 1,
                  1 if gathered else 0], np.int64).tofile(f)
        np.array([gamma, eps, rho, tau, 1.0 / N], np.float32).tofile(f)
        matrix(img, ld_img).tofile(f)
        matrix(txt, ld_txt).tofile(f)
        idx.astype(np.int64).tofile(f)
        u0i.tofile(f)
        u0t.tofile(f)
        if version == V2:
            t_img.tofile(f)
            t_txt.tofile(f)
        if gathered:
            glob["u_img"].tofile(f)
            glob["u_txt"].tofile(f)
            if version == V2:
                glob["tau_img"].tofile(f)
                glob["tau_txt"].tofile(f)
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0", TSAN_OPTIONS="report_thread_leaks=0", EMU_FETCHES="1")
    if SANITIZER == "memory":
        env["EMU_UNINIT"] = "1"
    r = subprocess.run([exe, fin, fout], capture_output=True, text=True, timeout=600, env=env)
    (tmp_path / "case.err").write_text(r.stderr)
    assert r.returncode == 0 and "Sanitizer" not in r.stderr, \
        "the CPU build of the kernels failed (sanitizer report below)\n" + r.stderr[:6000]
    out = np.fromfile(fout, np.float32)
    fields = [("d_img", b * d), ("d_txt", b * d), ("loss", 1)]
    if version in (V0, V3):
        fields.append(("d_tau", 1))
    if version == V2:
        fields += [("d_tau_img", b), ("d_tau_txt", b)]
    fields += [("g_img", b), ("g_txt", b), ("u_new_img", b), ("u_new_txt", b), ("u_img", N), ("u_txt", N)]
    got, p = {}, 0
    for k, n in fields:
        got[k] = out[p:p + n].astype(np.float64)
        p += n
    assert p == out.size
    ui, ut = u0i.astype(np.float64), u0t.astype(np.float64)
    kw = {}
    if gathered:
        kw = dict(u_glob_img=glob["u_img"].astype(np.float64), u_glob_txt=glob["u_txt"].astype(np.float64))
        if version == V2:
            kw.update(tau_glob_img=glob["tau_img"].astype(np.float64), tau_glob_txt=glob["tau_txt"].astype(np.float64))
    want = fcco_step(img.astype(np.float64), txt.astype(np.float64), off, b, idx, ui, ut, version=version, gamma=gamma,
                     eps=eps, rho=rho, tau=float(np.float32(tau)), tau_img=t_img.astype(np.float64),
                     tau_txt=t_txt.astype(np.float64), tau_grad_scale=1.0 / N, **kw)
    tol = 2e-2 if dtype == "bf16" else 1e-5
    errs = {}
    for k in ("d_img", "d_txt"):
        errs[k] = np.max(np.abs(got[k].reshape(b, d) - want[k])) / np.max(np.abs(want[k]))
    for k in ("g_img", "g_txt", "u_new_img", "u_new_txt"):
        errs[k] = np.max(np.abs(got[k] - want[k]) / np.abs(want[k]))
    errs["loss"] = abs(got["loss"][0] - want["loss"]) / want["loss_abs"]
    if version in (V0, V3):
        errs["d_tau"] = abs(got["d_tau"][0] - want["d_tau"]) / want["d_tau_abs"]
    if version == V2:
        for k in ("d_tau_img", "d_tau_txt"):
            errs[k] = np.max(np.abs(got[k] - want[k])) / np.max(np.abs(want[k]))
    # the state: the oracle's arrays after the step, everywhere (untouched entries bit for bit)
    mask = np.ones(N, bool)
    mask[idx] = False
    assert np.array_equal(got["u_img"][mask], u0i[mask].astype(np.float64))
    assert np.array_equal(got["u_txt"][mask], u0t[mask].astype(np.float64))
    errs["u_img"] = np.max(np.abs(got["u_img"][idx] - ui[idx]) / ui[idx])
    errs["u_txt"] = np.max(np.abs(got["u_txt"][idx] - ut[idx]) / ut[idx])
    bad = {k: v for k, v in errs.items() if not v <= tol}
    assert not bad, bad
    # per launch: direct-to-LDS loads (one per lane) and the lines of memory that the XCDs' L2 caches fetch for them
    return [(int(n), int(m)) for n, m in re.findall(r"loads (\d+) lines (\d+)", r.stderr)]


CASES = [
    # fp32 accuracy path: rows that are no 16-byte words (everything through registers); whole stages, the whole batch
    # local; a ragged last stage behind a whole one; rows padded to words, two strips; few pairs in plain loops, plain and gathered
    dict(B=37, b=11, off=13, d=19, version=V2, dtype="f32", ld_img=23),
    dict(B=64, b=64, off=0, d=64, version=V2, dtype="f32"),
    dict(B=66, b=66, off=0, d=36, version=V3, dtype="f32"),
    dict(B=130, b=70, off=33, d=68, version=V0, dtype="f32", ld_img=72),
    dict(B=16, b=5, off=9, d=30, version=V3, dtype="f32", ld_img=33),
    dict(B=23, b=6, off=11, d=70, version=V2, dtype="f32", gathered=True),
    # MFMA path, every tile ragged: guarded strip tiles on the ring (rows replaced by the last one), ragged last stage,
    # contraction with a guarded tail, fused state phase in the fold; padding between the rows of one side
    dict(B=300, b=140, off=100, d=72, version=V3, ld_img=80, flags=fc.TILES_256),
    dict(B=40, b=40, off=0, d=16, version=V0, flags=fc.TILES_256),
    # whole tiles: the persistent eight-wave strip kernel and the contraction's ring, next to a ragged anchor tile
    dict(B=512, b=300, off=212, d=128, version=V2, flags=fc.TILES_256),
    # the whole batch local, similarity matrix formed once on ragged tiles (column pass of the guarded kernel)
    dict(B=300, b=300, off=0, d=72, version=V2, flags=fc.SINGLE_PASS),
    # ... and on whole tiles (column pass of the persistent kernel)
    dict(B=512, b=512, off=0, d=128, version=V3, flags=fc.SINGLE_PASS),
    # contrast side over every global anchor (second strip, remote fold), ragged and on whole tiles (the persistent kernel)
    dict(B=300, b=100, off=50, d=72, version=V2, gathered=True, flags=fc.TILES_256),
    dict(B=512, b=256, off=256, d=128, version=V3, gathered=True, flags=fc.TILES_256),
    # ... on the small tiles, the library's own choice (pairs of contrast tiles, second strip added in the contraction)
    dict(B=300, b=100, off=50, d=72, version=V2, gathered=True),
    # 128 x 128 tiles, the library's own choice for a small batch: ragged everywhere with a guarded last stage; whole stages on the ring with rows replaced;
    # the whole batch local with a width below one stage; several splits with the finalize kernel
    dict(B=300, b=140, off=100, d=72, version=V3, ld_txt=80),
    dict(B=512, b=300, off=212, d=128, version=V2, flags=fc.TILES_128),
    dict(B=257, b=257, off=0, d=8, version=V0, flags=fc.TILES_128),
    dict(B=5120, b=64, off=640, d=64, version=V1, flags=fc.TILES_128),
    # fine tiles (opt-in): one split with the output tiles finished in place, and several splits with the finalize kernel
    dict(B=300, b=140, off=100, d=72, version=V3, flags=fc.FINE_TILES, ld_txt=80),
    dict(B=5120, b=64, off=640, d=64, version=V1, flags=fc.FINE_TILES),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join("%s%s" % (k, v) for k, v in c.items()))
def test_step_of_the_host_built_kernels_matches_the_oracle_under_asan(emu_step, tmp_path, case):
    run_case(emu_step, tmp_path, **case)


# Kernels that the library's plans keep for larger shapes than the emulation has time for: the plan is forced (build_emu.PLAN_RULES)
FORCED = [
    # small tiles: contraction on 128 x 128 output tiles behind the fold, with and without splits; strips of two workgroups
    # per compute unit with it; strips of 128 anchors and output tiles of 128 rows; splits of either row count; with gathered state
    dict(plan=dict(WIDE=1, NSPLIT=1), B=300, b=140, off=100, d=72, version=V2, ld_txt=80),
    dict(plan=dict(WIDE=1, NSPLIT=3), B=257, b=257, off=0, d=40, version=V3),
    dict(plan=dict(WIDE=1, WIDE_STRIPS=1), B=300, b=140, off=100, d=72, version=V0, ld_txt=80),
    dict(plan=dict(OUT_ROWS=128, NARROW=0), B=200, b=140, off=33, d=72, version=V2),
    dict(plan=dict(OUT_ROWS=32), B=200, b=140, off=33, d=72, version=V2, ld_img=80),
    dict(plan=dict(FEW=0), B=200, b=140, off=33, d=200, version=V2, ld_img=208),              # strips of 64 anchors
    dict(plan=dict(FEW=0, OWN_PREP=0), B=200, b=140, off=33, d=72, version=V3),
    dict(plan=dict(OWN_PREP=0), B=200, b=140, off=33, d=200, version=V0),                     # of 32, prepared by the launch before
    dict(plan=dict(OUT_ROWS=64), B=600, b=530, off=70, d=24, version=V3),
    dict(plan=dict(OUT_ROWS=64, NSPLIT=3, OWN_PREP=0), B=200, b=70, off=129, d=136, version=V0),
    dict(plan=dict(OUT_ROWS=128, NSPLIT=2), B=200, b=140, off=33, d=72, version=V3),
    dict(plan=dict(OUT_ROWS=64, NSPLIT=2, NARROW=0), B=200, b=140, off=33, d=72, version=V3, gathered=True),
    # large tiles: output tiles of the contraction of either width, a whole one and one cut short, on the ring and behind it
    dict(plan=dict(OUT_COLS=256), B=520, b=200, off=112, d=264, version=V1, flags=fc.TILES_256, ld_txt=272),
    dict(plan=dict(OUT_COLS=192), B=520, b=200, off=112, d=264, version=V2, flags=fc.TILES_256, ld_txt=272),
    # ... with gathered state, where the loop over whole stages forms its operand from both strips, two or three splits
    dict(plan=dict(OUT_COLS=256), B=700, b=40, off=300, d=40, version=V2, flags=fc.TILES_256, gathered=True),
    dict(plan=dict(OUT_COLS=192), B=520, b=200, off=112, d=264, version=V3, flags=fc.TILES_256, gathered=True, ld_txt=272),
    # fp32 path: 64 x 64 tiles of strips and gradients, splits, the single pass on them; splits with gathered state; one partial
    # sum over several tiles, as where the strips alone fill the static array
    dict(plan=dict(F32_TILES=1, GRAD_TILE=64, NSPLIT=2), B=150, b=70, off=33, d=68, ld_img=72, version=V3, dtype="f32"),
    dict(plan=dict(F32_TILES=1, GRAD_TILE=64), B=70, b=70, off=0, d=64, version=V2, dtype="f32"),
    dict(plan=dict(NSPLIT=3), B=130, b=40, off=70, d=128, version=V2, dtype="f32", gathered=True),
    dict(plan=dict(STATIC_BYTES=60000), B=70, b=70, off=0, d=36, version=V2, dtype="f32"),
]


@pytest.mark.parametrize("case", FORCED, ids=lambda c: "-".join("%s%s" % (k, v) for k, v in c.items()))
def test_plans_of_larger_shapes_on_the_host_built_kernels(emu_step, tmp_path, monkeypatch, case):
    for k, v in case["plan"].items():
        monkeypatch.setenv("EMU_" + k, str(v))
    run_case(emu_step, tmp_path, **{k: v for k, v in case.items() if k != "plan"})


def test_large_tile_contraction_shares_its_operands_inside_an_xcd(emu_step, tmp_path):
    """Three splits of two row tiles and two sides: the workgroups of an XCD read the same slice of the depth, so that the
    eight L2 caches together fetch little more than every line of the strips and the matrices once."""
    b, B, d = 260, 768, 72
    launches = run_case(emu_step, tmp_path, B=B, b=b, off=300, d=d, version=V3, flags=fc.TILES_256)
    contraction = launches[-2]                                     # the finalize kernel is the last
    strips, matrices = 2 * 512 * B * 2 // 128, 2 * B * d * 2 // 128
    assert strips < contraction[1] <= strips + matrices, (launches, strips, matrices)


@pytest.mark.parametrize("stages,cols", [(1, 256), (2, 192), (3, 256), (5, 192), (6, 256), (7, 256), (7, 192), (9, 256)])
def test_gathered_contraction_takes_any_run_of_stages(emu_step, tmp_path, monkeypatch, stages, cols):
    """Large tiles with gathered state: however many whole stages of 32 rows there are, few or an odd number, they go through the
    loop that keeps direct-to-LDS loads of X in flight, and the outputs agree with the oracle."""
    monkeypatch.setenv("EMU_OUT_COLS", str(cols))
    launches = run_case(emu_step, tmp_path, B=32 * stages + 1, b=9, off=7, d=cols, version=V2 if stages % 2 else V3,
                        flags=fc.TILES_256, gathered=True, N=300)
    assert launches[-2][0] >= 2 * stages * 32 * cols // 8, launches      # two sides, 8 elements per lane


@pytest.mark.parametrize("seed", range(8))
def test_random_small_shapes_on_the_host_built_kernels(emu_step, tmp_path, seed):
    """Shapes, strides, version and path drawn at random (seeded): B up to 300, any b and off, widths of 8 .. 320 that are
    no whole stages, padded rows; tile size asked for or left to the library, fine tiles, single pass, gathered state."""
    import random
    rng = random.Random(1000 + seed)
    B = rng.choice([rng.randint(2, 40), rng.randint(41, 300), 256])
    full = rng.random() < 0.3
    b = B if full else rng.randint(1, B)
    off = 0 if full else rng.randint(0, B - b)
    d = 8 * rng.choice([1, 2, 3, 4, 8, 9, 16, 17, 24, 32, 33, 40])
    path = ["256", "128", "auto", "fine", "single", "gathered", "128", "256"][seed]
    flags = {"256": fc.TILES_256, "128": fc.TILES_128, "auto": 0, "fine": fc.FINE_TILES, "single": fc.SINGLE_PASS,
             "gathered": fc.TILES_256}[path]
    if path == "single":
        b, off = B, 0
    run_case(emu_step, tmp_path, B=B, b=b, off=off, d=d, version=rng.randint(0, 3), flags=flags,
             N=max(b, 50) + rng.randint(0, 500), ld_img=d + 8 * rng.randint(0, 2), ld_txt=d + 8 * rng.randint(0, 2),
             seed=77 + seed, gathered=(path == "gathered"))


# ------------------------------------------------------------------ the step with the temperature update fused in
UPD = dict(lr=2e-3, step=3, beta1=0.9, beta2=0.98, eps=1e-8, tau_min=0.02, lr_drop_below=0.06, lr_drop_factor=1.0 / 3.0)


@pytest.mark.parametrize("case", [
    # V2 on records {u_1, tau_1, m_1, v_1, u_2, tau_2, m_2, v_2} that the state kernel moves as 16-byte words per side
    dict(B=300, b=140, off=100, d=72, version=V2, optimizer=ADAMW, stride=8, flags=fc.TILES_256),
    # ... records with four floats of padding that must stay untouched; the state phase inside the fold (small tiles)
    dict(B=300, b=140, off=100, d=72, version=V2, optimizer=ADAMW, stride=12),
    # dense arrays, field by field; without a second moment, whose arrays nothing may touch then (emu_main.cpp): anchors finished
    # by workgroups of their own, by those of the output tiles, by k_state and by the fold
    dict(B=40, b=40, off=0, d=16, version=V2, optimizer=LION, stride=1),
    dict(plan=dict(OUT_ROWS=32, FINISHERS=0), B=140, b=70, off=33, d=40, version=V2, optimizer=LION, stride=1),
    dict(plan=dict(FUSED=0), B=140, b=70, off=33, d=40, version=V2, optimizer=SGDM, stride=1),
    dict(B=140, b=70, off=33, d=40, version=V2, optimizer=SGDM, stride=1, flags=fc.TILES_256),
    # the global temperature stepped by a kernel of its own once its gradient is complete
    dict(B=300, b=140, off=100, d=72, version=V3, optimizer=ADAMW, stride=1),
], ids=lambda c: "-".join("%s%s" % (k, v) for k, v in c.items()))
def test_step_with_temperature_update_of_the_host_built_kernels(emu_step, tmp_path, monkeypatch, case):
    """fastclip_step_update_tau: every output of the step, the state, and the temperatures with their moments after
    Proc. temperature_update, against the oracle's step followed by its temperature update."""
    for k, v in case.get("plan", {}).items():
        monkeypatch.setenv("EMU_" + k, str(v))
    B, b, off, d, version, S = case["B"], case["b"], case["off"], case["d"], case["version"], case["stride"]
    N, gamma, eps, rho, tau = max(700, b + 100), 0.6, 1e-6, 6.5, 0.07
    rng = np.random.default_rng(5)
    img, txt = make_embeddings(51, B, d, 0.5, "bf16")
    idx = draw_indices(52, b, N)
    f32 = lambda a: np.asarray(a, np.float32)
    st = dict(u_img=f32(np.where(rng.random(N) < 0.5, 0.0, rng.uniform(0.05, 2.0, N))),
              u_txt=f32(np.where(rng.random(N) < 0.5, 0.0, rng.uniform(0.05, 2.0, N))),
              tau_img=f32(rng.uniform(0.04, 0.1, N)), tau_txt=f32(rng.uniform(0.04, 0.1, N)),
              m_img=f32(rng.normal(0, 0.1, N)), v_img=f32(rng.uniform(0.0, 0.05, N)),
              m_txt=f32(rng.normal(0, 0.1, N)), v_txt=f32(rng.uniform(0.0, 0.05, N)))
    m0, v0 = np.float32(0.03), np.float32(0.002)
    fin, fout = str(tmp_path / "case.in"), str(tmp_path / "case.out")
    with open(fin, "wb") as f:
        np.array([version, fc.BF16, case.get("flags", 0), B, b, off, d, d, d, N, S, 0], np.int64).tofile(f)
        np.array([gamma, eps, rho, tau, 1.0 / N], np.float32).tofile(f)
        bf16_bits(img).tofile(f)
        bf16_bits(txt).tofile(f)
        idx.astype(np.int64).tofile(f)
        st["u_img"].tofile(f)
        st["u_txt"].tofile(f)
        if version == V2:
            st["tau_img"].tofile(f)
            st["tau_txt"].tofile(f)
        np.array([case["optimizer"], UPD["step"]], np.int64).tofile(f)
        np.array([UPD["lr"], UPD["beta1"], UPD["beta2"], UPD["eps"], UPD["tau_min"], UPD["lr_drop_below"],
                  UPD["lr_drop_factor"]], np.float32).tofile(f)
        if version == V2:
            for k in ("m_img", "v_img", "m_txt", "v_txt"):
                st[k].tofile(f)
        else:
            np.array([m0], np.float32).tofile(f)
            np.array([v0], np.float32).tofile(f)
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0", TSAN_OPTIONS="report_thread_leaks=0")
    r = subprocess.run([emu_step, fin, fout, "tau"], capture_output=True, text=True, timeout=600, env=env)
    assert r.returncode == 0 and "Sanitizer" not in r.stderr, r.stderr[:6000]
    out = np.fromfile(fout, np.float32).astype(np.float64)
    fields = [("d_img", b * d), ("d_txt", b * d), ("loss", 1)]
    fields += [("d_tau", 1)] if version != V2 else [("d_tau_img", b), ("d_tau_txt", b)]
    fields += [("g_img", b), ("g_txt", b), ("u_new_img", b), ("u_new_txt", b), ("u_img", N), ("u_txt", N)]
    fields += [(k, N) for k in ("tau_img", "tau_txt", "m_img", "v_img", "m_txt", "v_txt")] if version == V2 else \
              [("tau", 1), ("m", 1), ("v", 1)]
    got, p = {}, 0
    for k, n in fields:
        got[k] = out[p:p + n]
        p += n
    assert p == out.size
    # the oracle: the step with the temperatures of before the call, then the temperature update from its gradients
    w = {k: v.astype(np.float64) for k, v in st.items()}
    want = fcco_step(img.astype(np.float64), txt.astype(np.float64), off, b, idx, w["u_img"], w["u_txt"], version=version,
                     gamma=gamma, eps=eps, rho=rho, tau=float(np.float32(tau)), tau_img=w["tau_img"].copy(),
                     tau_txt=w["tau_txt"].copy(), tau_grad_scale=1.0 / N)
    kw = {k: (float(np.float32(v)) if isinstance(v, float) else v) for k, v in UPD.items()}
    if version == V2:
        temperature_update(V2, want, optimizer=case["optimizer"], tau_img=w["tau_img"], tau_txt=w["tau_txt"], idx=idx,
                           m_img=w["m_img"], v_img=w["v_img"], m_txt=w["m_txt"], v_txt=w["v_txt"], **kw)
        for k in ("tau_img", "tau_txt", "m_img", "v_img", "m_txt", "v_txt"):
            if case["optimizer"] in (LION, SGDM) and k.startswith("v_"):
                assert np.array_equal(got[k], st[k].astype(np.float64))          # they keep no second moment
                continue
            scale = np.max(np.abs(w[k]))
            assert np.max(np.abs(got[k] - w[k])) <= 2e-2 * scale, k
            mask = np.ones(N, bool)
            mask[idx] = False
            assert np.array_equal(got[k][mask], st[k][mask].astype(np.float64)), k    # other samples untouched
    else:
        t_new, m_new, v_new = temperature_update(version, want, optimizer=case["optimizer"], tau=float(np.float32(tau)),
                                                 m=float(m0), v=float(v0), **kw)
        assert got["tau"][0] == pytest.approx(t_new, rel=1e-4)
        assert got["m"][0] == pytest.approx(m_new, rel=2e-2) and got["v"][0] == pytest.approx(v_new, rel=4e-2)
    for k in ("d_img", "d_txt"):
        assert np.max(np.abs(got[k].reshape(b, d) - want[k])) <= 2e-2 * np.max(np.abs(want[k])), k
    for k in ("g_img", "g_txt", "u_new_img", "u_new_txt"):
        assert np.max(np.abs(got[k] - want[k]) / np.abs(want[k])) <= 2e-2, k
    assert np.max(np.abs(got["u_img"] - w["u_img"])) <= 2e-2 * np.max(w["u_img"])
    assert np.max(np.abs(got["u_txt"] - w["u_txt"])) <= 2e-2 * np.max(w["u_txt"])


# ------------------------------------------------------------------ the small entry points
@pytest.mark.parametrize("b,d,n,pads", [(37, 19, 300, (3, 5)), (5, 4104, 2, (3, 5)), (130, 72, 1, (3, 5)), (1, 1, 1000, (3, 5)),
                                        (37, 72, 3, (4, 8)), (9, 1024, 3, (0, 0)), (5, 1028, 3, (0, 4))])
def test_small_entry_points_of_the_host_built_kernels(emu_step, tmp_path, b, d, n, pads):
    """fastclip_normalize_rows (a wavefront per row, padded rows on both sides; whole groups of four elements up to a width of
    1024, and behind it), fastclip_check_indices (hash table on
    the device; distinct indices pass, a repeated one is reported), fastclip_state_update (Eq. 1 alone)."""
    rng = np.random.default_rng(b + d)
    ld_raw, ld_unit, N = d + pads[0], d + pads[1], 4 * n + 7
    raw = np.full((b, ld_raw), np.nan, np.float32)
    raw[:, :d] = rng.normal(0, 1, (b, d)) * rng.uniform(0.1, 30.0, (b, 1))
    idx = draw_indices(9, n, N)
    sums = [rng.uniform(1.0, 50.0, n).astype(np.float32) for _ in range(2)]
    u0 = [np.where(rng.random(N) < 0.5, 0.0, rng.uniform(0.05, 2.0, N)).astype(np.float32) for _ in range(2)]
    gamma, M = np.float32(0.3), np.float32(77.0)
    fin, fout = str(tmp_path / "misc.in"), str(tmp_path / "misc.out")
    with open(fin, "wb") as f:
        np.array([b, d, ld_raw, ld_unit, N, n], np.int64).tofile(f)
        np.array([gamma, M], np.float32).tofile(f)
        raw.reshape(-1)[: (b - 1) * ld_raw + d].tofile(f)
        idx.astype(np.int64).tofile(f)
        for a in sums + u0:
            a.tofile(f)
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0", TSAN_OPTIONS="report_thread_leaks=0")
    r = subprocess.run([emu_step, "misc", fin, fout], capture_output=True, text=True, timeout=600, env=env)
    assert r.returncode == 0 and "Sanitizer" not in r.stderr, r.stderr[:6000]
    blob = open(fout, "rb").read()
    n_unit = (b - 1) * ld_unit + d
    norm = np.frombuffer(blob, np.float32, b, 0).astype(np.float64)
    bits = np.frombuffer(blob, np.uint16, n_unit, 4 * b)
    st = np.frombuffer(blob, np.int32, 2, 4 * b + 2 * n_unit)
    rest = np.frombuffer(blob, np.float32, 2 * N + 2 * n, 4 * b + 2 * n_unit + 8).astype(np.float64)
    want_unit, want_norm = normalize_rows(raw[:, :d])
    assert np.max(np.abs(norm - want_norm) / want_norm) <= 1e-6
    full = np.zeros(b * ld_unit, np.uint16)
    full[:n_unit] = bits
    unit = (full.reshape(b, ld_unit)[:, :d].astype(np.uint32) << 16).view(np.float32).astype(np.float64)
    assert np.max(np.abs(unit - want_unit)) <= 2.0 ** -8                       # one rounding to bf16 of values <= 1
    assert st[0] == fc.OK and st[1] == (fc.ERR_INDEX if n > 1 else fc.OK)
    u_img, u_txt, new_img, new_txt = rest[:N], rest[N:2 * N], rest[2 * N:2 * N + n], rest[2 * N + n:]
    for got, got_new, u_before, s_ in ((u_img, new_img, u0[0], sums[0]), (u_txt, new_txt, u0[1], sums[1])):
        want = u_before.astype(np.float64)
        new = ema_update(want, idx, s_.astype(np.float64) / float(M), float(gamma))
        assert np.max(np.abs(got - want) / np.maximum(want, 1e-30)) <= 1e-6
        assert np.max(np.abs(got_new - new) / new) <= 1e-6


# ------------------------------------------------------------------ what the single pass rounds
def bf16_round(x):
    """Nearest bf16, ties to even, as fp64."""
    u = np.ascontiguousarray(x, np.float32).view(np.uint32)
    return (((u + 0x7fff + ((u >> 16) & 1)) & 0xffff0000).astype(np.uint32)).view(np.float32).astype(np.float64)


@pytest.mark.parametrize("b,d", [(300, 72), (512, 64)])
def test_single_pass_rounds_each_side_s_weights_divided_by_its_own_coefficient(emu_step, tmp_path, b, d):
    """The whole batch local, similarity matrix formed once: either side's contraction takes w / c_own as bf16, w = c1_r l1 + c2_q l2,
    and multiplies by c_own in fp32, as the two-strip form does.  Taken as bf16 themselves, the weights w would be rounded
    elsewhere and the gradients would move by 1.6e-3 of an operand's size per product.

    Tolerance: a fourth of the distance between those two forms here.  What is left between this model in fp64 and the kernels
    are single elements that the fp32 evaluation rounds to the other bf16 neighbour: the exponentials are off by some 3e-6 (an
    exponent of up to 60 in fp32), so one in a thousand of them and of the weights, 4e-3 each: 1.3e-4 per product against 1.6e-3."""
    run_case(emu_step, tmp_path, B=b, b=b, off=0, d=d, version=V2, flags=fc.SINGLE_PASS)
    raw, n_state = open(tmp_path / "case.in", "rb").read(), 900
    eps = float(np.frombuffer(raw, np.float32, 5, 96)[1])
    at, rows = 96 + 20, []
    for _ in range(2):
        bits = np.frombuffer(raw, np.uint16, b * d, at).reshape(b, d).astype(np.uint32)
        rows.append((bits << 16).view(np.float32).astype(np.float64))
        at += 2 * b * d
    idx = np.frombuffer(raw, np.int64, b, at)
    at += 8 * b + 8 * n_state                                                # u_img, u_txt
    tau = [np.frombuffer(raw, np.float32, n_state, at + 4 * n_state * k)[idx].astype(np.float64) for k in range(2)]
    out = np.fromfile(tmp_path / "case.out", np.float32).astype(np.float64)
    got = [out[:b * d].reshape(b, d), out[b * d:2 * b * d].reshape(b, d)]
    at = 2 * b * d + 1 + 2 * b                                               # loss, d_tau_img, d_tau_txt
    g, u = [out[at + k * b:at + (k + 1) * b] for k in (0, 1)], [out[at + k * b:at + (k + 1) * b] for k in (2, 3)]

    M = b - 1.0
    c = [1.0 / (b * M * (eps + u[k])) for k in (0, 1)]
    s = rows[0] @ rows[1].T                                                  # [image][text]
    off_diagonal = ~np.eye(b, dtype=bool)
    l1 = bf16_round(np.exp((s - np.diag(s)[:, None]) / tau[0][:, None]) * off_diagonal)
    l2 = bf16_round(np.exp((s - np.diag(s)[None, :]) / tau[1][None, :]) * off_diagonal)      # of text q against image r, at [r][q]
    w = c[0][:, None] * l1 + c[1][None, :] * l2
    diagonal = (c[0] * M * g[0] + c[1] * M * g[1])[:, None]
    one = bf16_round(w)
    for side, (weights, other, whole) in enumerate(((w / c[0][:, None], rows[1], one), ((w / c[1][None, :]).T, rows[0], one.T))):
        want = c[side][:, None] * (bf16_round(weights) @ other) - diagonal * other
        distance = np.linalg.norm(whole @ other - diagonal * other - want)
        assert np.linalg.norm(got[side] - want) <= distance / 4, (side, np.linalg.norm(got[side] - want), distance)


# ------------------------------------------------------------------ one array for both sides' temperatures
@pytest.mark.parametrize("b,optimizer,shared", [
    # nothing shared; one temperature for both sides with its moments; a moment shared alone; a second moment that is not kept
    (70, ADAMW, 0), (70, ADAMW, 7), (300, SGDM, 3), (70, SGDM, 2), (70, ADAMW, 4), (70, LION, 4)])
def test_temperature_update_with_arrays_that_both_sides_share(emu_step, tmp_path, monkeypatch, b, optimizer, shared):
    """fastclip_temperature_update (V2) where an array is passed for both sides: an anchor's image step comes first and its text
    step goes on from there, in whatever order the workgroups run (last first here)."""
    monkeypatch.setenv("EMU_BACKWARDS", "1")
    N, step = 2 * b, 3
    rng = np.random.default_rng(b + shared)
    f32 = lambda lo, hi, n: rng.uniform(lo, hi, n).astype(np.float32)
    idx = draw_indices(60, b, N)
    g = [f32(-1, 1, b) for _ in range(2)]
    given = [[f32(0.05, 0.1, N), f32(-0.1, 0.1, N), f32(0.01, 0.05, N)] for _ in range(2)]        # tau, m, v of either side
    hp = [float(np.float32(x)) for x in (2e-3, 0.9, 0.98, 1e-6)]
    fin, fout = str(tmp_path / "tau.in"), str(tmp_path / "tau.out")
    with open(fin, "wb") as f:
        np.array([b, N, optimizer, step, shared], np.int64).tofile(f)
        np.array(hp, np.float32).tofile(f)
        for a in [idx.astype(np.int64)] + g + given[0] + given[1]:
            a.tofile(f)
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0", TSAN_OPTIONS="report_thread_leaks=0")
    r = subprocess.run([emu_step, "temperatures", fin, fout], capture_output=True, text=True, timeout=600, env=env)
    assert r.returncode == 0 and "Sanitizer" not in r.stderr, r.stderr[:6000]
    got = np.fromfile(fout, np.float32).astype(np.float64).reshape(2, 3, N)
    want = [[a.astype(np.float64) for a in side] for side in given]
    for k in range(3):
        if shared >> k & 1:
            want[1][k] = want[0][k]
    keeps_v = optimizer == ADAMW
    temperature_update(V2, dict(d_tau_img=g[0].astype(np.float64), d_tau_txt=g[1].astype(np.float64)), optimizer=optimizer, lr=hp[0],
                       step=step, beta1=hp[1], beta2=hp[2], eps=hp[3], idx=idx,
                       **{n + s: (want[i][k] if n != "v_" or keeps_v else want[i][k].copy())
                          for i, s in ((0, "img"), (1, "txt")) for k, n in enumerate(("tau_", "m_", "v_"))})
    # a dozen fp32 operations a step, each rounded once: 2^-24 of what they add up to, which is about 2 at most
    for side in range(2):
        for k in range(3):
            assert np.max(np.abs(got[side][k] - want[side][k])) <= 16 * 2.0 ** -24, (side, k)


# ------------------------------------------------------------------ which kernels a plan launches
def launches_of(tmp_path):
    """(workgroups, threads) of every launch of the step that run_case has run."""
    return [(int(w), int(t)) for w, t in re.findall(r"workgroups (\d+) threads (\d+)", (tmp_path / "case.err").read_text())]


@pytest.mark.parametrize("case,prep,state", [
    # the whole batch local, ragged tiles; two strips, rows that begin inside the batch, several splits of the gradients
    (dict(B=40, b=40, off=0, d=20, version=V3), 0, 0),
    (dict(plan=dict(F32_OWN_PREP=0), B=40, b=40, off=0, d=20, version=V3), 1, 0),
    (dict(plan=dict(GRAD_STATE=0), B=40, b=40, off=0, d=20, version=V2), 0, 1),
    (dict(plan=dict(F32_OWN_PREP=0, GRAD_STATE=0), B=40, b=40, off=0, d=20, version=V0), 1, 1),
    (dict(plan=dict(NSPLIT=2, F32_OWN_PREP=0), B=70, b=36, off=33, d=20, version=V0), 1, 0),
    (dict(plan=dict(NSPLIT=2, GRAD_STATE=0), B=70, b=36, off=33, d=20, ld_img=23, version=V3), 0, 1),
    # wide rows of a whole local batch, which the rule leaves to the launch before the strips
    (dict(B=28, b=28, off=0, d=516, version=V2), 1, 0),
    (dict(plan=dict(F32_OWN_PREP=1), B=28, b=28, off=0, d=516, ld_img=519, version=V2), 0, 0),
    # gathered state is prepared by the launch before, whose gradients run the state phase all the same
    (dict(B=60, b=20, off=11, d=20, version=V2, gathered=True), 1, 0),
    (dict(plan=dict(GRAD_STATE=0), B=60, b=20, off=11, d=20, version=V2, gathered=True), 1, 1),
], ids=lambda c: "-".join("%s%s" % (k, v) for k, v in c.items()) if isinstance(c, dict) else "")
def test_f32_launches_with_and_without_prep_and_state_phase(emu_step, tmp_path, monkeypatch, case, prep, state):
    """The fp32 path's strips prepare their anchors and its gradients run the state phase, or launches of 256 threads before and
    between them do: the launches are those that the plan promises, and the outputs the oracle's either way."""
    for k, v in case.get("plan", {}).items():
        monkeypatch.setenv("EMU_" + k, str(v))
    run_case(emu_step, tmp_path, dtype="f32", **{k: v for k, v in case.items() if k != "plan"})
    threads = [t for _, t in launches_of(tmp_path)]
    assert threads == [256] * prep + [512] + [256] * state + [512], threads


@pytest.mark.parametrize("plan,anchors", [({}, 32), (dict(FEW=0), 64), (dict(FEW=0, NARROW=0), 128)])
def test_anchors_of_a_small_strip_tile(emu_step, tmp_path, monkeypatch, plan, anchors):
    """Strips of the small tiles, the launch before the contraction: two contrast tiles, 130 anchors in tiles of 32 (one round of
    workgroups, the library's own choice here), 64 and 128, two strips."""
    for k, v in plan.items():
        monkeypatch.setenv("EMU_" + k, str(v))
    run_case(emu_step, tmp_path, B=200, b=130, off=33, d=40, version=V3)
    launches = launches_of(tmp_path)
    assert launches[0] == (2 * 2 * -(-130 // anchors), 512), launches
