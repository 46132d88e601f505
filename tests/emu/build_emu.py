"""Builds the CPU emulation of libfastclip: the library's own sources compiled for the host against the stand-in
hip/hip_runtime.h of this folder, linked with emu_main.cpp into _build/emu/emu_step, AddressSanitizer on.

The sources are copied with the few constructs a host compiler cannot take replaced by calls into the stand-in: inline
assembly (direct-to-LDS loads, accumulator reads) and the address-space attributes.  Indexing, guards, barriers and the
order of operations are the product's.  So that a small shape can run what the library's plans keep for large ones, the rules
in PLAN_RULES also listen to environment variables (EMU_...): unset, they decide as in the product."""
from __future__ import annotations

import os
import re
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))
CSRC = os.path.join(ROOT, "paper_2407_01445_amd", "csrc")
OUT = os.path.join(ROOT, "_build", "emu")
EXE = os.path.join(OUT, "emu_step")


def host_compiler():
    for c in ("/opt/rocm/llvm/bin/clang++", shutil.which("clang++")):
        if c and os.path.exists(c):
            return c
    return None


def _asm_replacement(m):
    t = m.group(0)
    if "s_add_u32 m0" in t:                      # 16 bytes per lane into LDS at (uniform + IMM) + 16 lane
        return "emu_dma(uniform_base, lane_byte_off, lds_uniform + (uint32_t)IMM, 16);"
    if "global_load_lds_dwordx4" in t:
        return "emu_dma(uniform_base, lane_byte_off, lds_byte_addr, 16);"
    if "global_load_lds_dword " in t:
        return "emu_dma(uniform_base, lane_byte_off, lds_byte_addr, 4);"
    if "s_load_dword" in t:                      # arguments into the scalar cache
        return "(void)w0, (void)w8;"
    if "v_accvgpr_read_b32" in t:
        return "x = in_agpr;"
    if re.search(r'asm volatile\(""', t):         # keeps a value alive, nothing to run
        return "(void)0;"
    raise RuntimeError("inline assembly the emulation does not know: " + t)


def _forced(expr, name, kind="atoi"):
    return '(getenv("%s") ? %s(getenv("%s")) : (%s))' % (name, kind, name, expr)


# (file, the product's text, what the emulation compiles instead); every text must be there, so that a rule that changes
# here fails loudly
PLAN_RULES = [
    # small tiles: rows of an output tile and splits of k_contract_t128_bf16; the 128 x 128 contraction; either kind of strips
    ("fastclip_api.hip", "  for (int64_t rows = L->gathered ? 64 : 32; rows <= (L->gathered ? 64 : 128); rows *= 2) {",
     '  for (int64_t rows = L->gathered ? 64 : 32; rows <= (L->gathered ? 64 : 128); rows *= 2) {\n'
     '    if (getenv("EMU_OUT_ROWS") && atoi(getenv("EMU_OUT_ROWS")) != rows) continue;'),
    ("fastclip_api.hip", "      if (best_cost == 0.0 || cost < best_cost) {",
     '      if (getenv("EMU_NSPLIT") && atoi(getenv("EMU_NSPLIT")) != ns) continue;\n'
     '      if (best_cost == 0.0 || cost < best_cost) {'),
    ("fastclip_api.hip", "    if (ns == 1 || cost < wide_cost) { split = ns; wide_cost = cost; }",
     '    if (getenv("EMU_NSPLIT") && atoi(getenv("EMU_NSPLIT")) != ns) continue;\n'
     '    if (wide_cost == 0.0 || cost < wide_cost) { split = ns; wide_cost = cost; }'),
    ("fastclip_api.hip", "  if (rounds < 2 || cfg.b < 448) return true;",
     '  if (getenv("EMU_WIDE") ? !atoi(getenv("EMU_WIDE")) : rounds < 2 || cfg.b < 448) return true;'),
    ("fastclip_api.hip", "  if (wgs >= (cfg.b > 512 ? 256 : 257) &&", '  if (getenv("EMU_WIDE") || wgs >= (cfg.b > 512 ? 256 : 257) &&'),
    ("fastclip_api.hip", "L->wide_strips = tiles > 256 && tiles < 512 && (4 * cfg.b > 3 * cfg.B || L->nparts % 2);",
     "L->wide_strips = " + _forced("tiles > 256 && tiles < 512 && (4 * cfg.b > 3 * cfg.B || L->nparts % 2)", "EMU_WIDE_STRIPS") + ";"),
    ("fastclip_api.hip", "L->own_prep = cfg.d <= (tiles <= 256 ? (rows <= 64 ? 1200 : 1400) : (tiles <= 512 ? 480 : 0));",
     "L->own_prep = " + _forced("cfg.d <= (tiles <= 256 ? (rows <= 64 ? 1200 : 1400) : (tiles <= 512 ? 480 : 0))", "EMU_OWN_PREP") + ";"),
    ("fc_internal.hpp", "return 2 * ((L.b + 63) / 64) * (int64_t)L.nparts <= 256;",
     "return " + _forced("2 * ((L.b + 63) / 64) * (int64_t)L.nparts <= 256", "EMU_NARROW") + ";"),
    ("fc_internal.hpp", "return 2 * ((L.b + 31) / 32) * (int64_t)L.nparts <= 256;",
     "return " + _forced("2 * ((L.b + 31) / 32) * (int64_t)L.nparts <= 256", "EMU_FEW") + ";"),
    # ... the state phase: inside the contraction or on its own; by workgroups of its own there or by those of the output tiles
    ("fastclip_api.hip", "const bool fused = r == 1 || (rows == 64 && nq <= 256 && L->nparts <= 64);",
     "const bool fused = " + _forced("r == 1 || (rows == 64 && nq <= 256 && L->nparts <= 64)", "EMU_FUSED") + ";"),
    ("kernels_tiles128.hip", "g.finishers = L.fused_state && groups + finishers <= 256 ? (int)finishers : 0;",
     "g.finishers = L.fused_state && " + _forced("groups + finishers <= 256", "EMU_FINISHERS") + " ? (int)finishers : 0;"),
    # large tiles: columns of an output tile of the contraction
    ("fastclip_api.hip", "      const double width = cols == 256 || L->gathered ? 1.0 : 0.80;",
     '      if (getenv("EMU_OUT_COLS") && atoi(getenv("EMU_OUT_COLS")) != cols) return;\n'
     '      const double width = cols == 256 || L->gathered ? 1.0 : 0.80;'),
    # fp32 path: tile sizes, plain loops, what is left of a plan that has to fit the static array
    ("fastclip_api.hip", "((cfg.B + 63) / 64) >= 256 ? 64 : 32;", "((cfg.B + 63) / 64) >= " + _forced("256", "EMU_F32_TILES") + " ? 64 : 32;"),
    ("fastclip_api.hip", "  for (int T = 32; T <= 64; T += 32) {",
     '  for (int T = 32; T <= 64; T += 32) {\n    if (getenv("EMU_GRAD_TILE") && atoi(getenv("EMU_GRAD_TILE")) != T) continue;'),
    # ... whether its strips prepare the anchors and its gradients run the state phase
    ("fastclip_api.hip", "L->own_prep = L->strip_tile == 32 && !L->gathered && (!L->square || cfg.d <= 512) && strip_wgs <= 512;",
     "L->own_prep = L->strip_tile == 32 && !L->gathered && " + _forced("(!L->square || cfg.d <= 512) && strip_wgs <= 512", "EMU_F32_OWN_PREP") + ";"),
    ("fastclip_api.hip", "    L->grad_state = room.state_rides && L->grad_tile == 32 &&",
     "    L->grad_state = " + _forced("1", "EMU_GRAD_STATE") + " && room.state_rides && L->grad_tile == 32 &&"),
    ("fastclip_api.hip", "  constexpr int64_t kLimit = FASTCLIP_STATIC_SCRATCH_BYTES;",
     "  const int64_t kLimit = " + _forced("FASTCLIP_STATIC_SCRATCH_BYTES", "EMU_STATIC_BYTES") + ";"),
]


def generate():
    gen = os.path.join(OUT, "gen")
    os.makedirs(gen, exist_ok=True)
    units = []
    for d, names in ((CSRC, sorted(os.listdir(CSRC))), (os.path.join(ROOT, "include"), ["fastclip.h"])):
        for n in names:
            if not n.endswith((".hip", ".hpp", ".h")):
                continue
            s = open(os.path.join(d, n)).read()
            s = s.replace("__attribute__((address_space(3)))", "").replace("__attribute__((address_space(1)))", "")
            s = re.sub(r'asm volatile\((?:[^;]|\n)*?\);', _asm_replacement, s)
            for name, text, instead in PLAN_RULES:
                if name == n:
                    if text not in s:
                        raise RuntimeError("%s: the rule has changed: %s" % (name, text))
                    s = s.replace(text, instead)
            out = os.path.join(gen, n.replace(".hip", ".inc"))
            open(out, "w").write(s)
            if n.endswith(".hip"):
                units.append(out)
    return gen, units


def build(sanitizer: str = "-fsanitize=address") -> str:
    cxx = host_compiler()
    if cxx is None:
        raise RuntimeError("no host clang++")
    gen, units = generate()
    obj = os.path.join(OUT, "obj")
    os.makedirs(obj, exist_ok=True)
    flags = ["-std=c++17", "-O1", "-g", "-fno-omit-frame-pointer", sanitizer, "-I", HERE, "-I", gen, "-pthread",
             "-Wno-unused-value", "-Wno-ignored-attributes"]

    def one(src):
        o = os.path.join(obj, os.path.basename(src).rsplit(".", 1)[0] + ".o")
        r = subprocess.run([cxx, *flags, "-x", "c++", "-c", src, "-o", o], capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError("host build of %s failed:\n%s" % (src, r.stderr[-4000:]))
        return o

    with ThreadPoolExecutor(max_workers=4) as ex:
        objs = list(ex.map(one, units + [os.path.join(HERE, "emu_main.cpp")]))
    r = subprocess.run([cxx, *flags, *objs, "-o", EXE], capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stderr[-4000:])
    return EXE


if __name__ == "__main__":
    import sys
    print(build(*sys.argv[1:2]))
