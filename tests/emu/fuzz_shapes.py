"""Random small shapes through the host build of the kernels (tests/emu) under AddressSanitizer, every path by random
flags, each compared with the oracle:  python tests/emu/fuzz_shapes.py <seed> <count>.  Not collected by pytest (the
seeded subset in tests/test_kernels_on_cpu.py is); about 7 s per case."""
import sys, pathlib, tempfile, time, random, traceback
import os
HERE = os.path.dirname(os.path.abspath(__file__))
for p in (os.path.dirname(os.path.dirname(HERE)), os.path.dirname(HERE), HERE):
    sys.path.insert(0, p)
import build_emu, test_kernels_on_cpu as t
from paper_2407_01445_amd import binding as fc
seed0 = int(sys.argv[1]); count = int(sys.argv[2])
exe = build_emu.build()
rng = random.Random(seed0)
fails = 0
for it in range(count):
    B = rng.choice([rng.randint(2, 40), rng.randint(41, 300), rng.randint(257, 700), rng.choice([256, 512, 768])])
    full = rng.random() < 0.3
    b = B if full else rng.randint(1, B)
    off = 0 if full else rng.randint(0, B - b)
    d = 8 * rng.choice([1, 2, 3, 4, 8, 9, 16, 17, 24, 32, 33, 40])
    version = rng.randint(0, 3)
    path = rng.choice(["256", "128", "auto", "fine", "single", "gathered", "f32"])
    flags = {"256": fc.TILES_256, "128": fc.TILES_128, "auto": 0, "fine": fc.FINE_TILES,
             "single": fc.SINGLE_PASS | (fc.TILES_256 if rng.random() < 0.5 else 0), "gathered": rng.choice([0, fc.TILES_256]), "f32": 0}[path]
    pad = 8
    if path == "f32":
        B, b, off, d, pad = B // 3 + 2, max(1, b // 3), off // 3, d // 4 + rng.randint(0, 3), rng.choice([1, 4])
    forced = {}
    if path in ("auto", "128") and rng.random() < 0.5:
        forced = rng.choice([dict(EMU_WIDE=1), dict(EMU_WIDE=1, EMU_WIDE_STRIPS=1), dict(EMU_OUT_ROWS=128, EMU_NARROW=0)])
    elif path == "f32" and rng.random() < 0.5:
        forced = dict(EMU_F32_TILES=1, EMU_GRAD_TILE=64)
    for k in ("EMU_WIDE", "EMU_WIDE_STRIPS", "EMU_OUT_ROWS", "EMU_NARROW", "EMU_F32_TILES", "EMU_GRAD_TILE"):
        os.environ.pop(k, None)
        if k in forced:
            os.environ[k] = str(forced[k])
    kw = dict(B=B, b=b, off=off, d=d, version=version, flags=flags, N=max(b, 50) + rng.randint(0, 500),
              ld_img=d + pad * rng.randint(0, 2), ld_txt=d + pad * rng.randint(0, 2), seed=seed0 * 1000 + it,
              gathered=(path == "gathered" or path == "f32" and rng.random() < 0.3), dtype="f32" if path == "f32" else "bf16")
    t0 = time.time()
    try:
        t.run_case(exe, pathlib.Path(tempfile.mkdtemp()), **kw)
        print("ok   %5.1fs %s %s" % (time.time() - t0, path, dict(kw, **forced)), flush=True)
    except Exception as e:
        fails += 1
        print("FAIL %5.1fs %s %s\n%s" % (time.time() - t0, path, dict(kw, **forced), str(e)[:3000]), flush=True)
print("done", count, "fails", fails)
