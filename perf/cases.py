"""Work that users of this library have it do: FCCO steps through the public entry points of `binding`, over the range of
batch sizes, widths, storage types and options that the step is made for.

A case is one worker's step: b local anchors (rows off .. off + b - 1) of a global batch of B pairs of width d.

    dtype     "bf16" (MFMA path) or "f32" (accuracy path): storage type of the embeddings
    version   0 .. 3: the temperature scheme (v0, v1, v3 one global temperature, v2 one per sample and side)
    ld        row stride of the embedding matrices, >= d
    N         samples in the per-sample state
    records   the state is one record of 8 floats per sample instead of separate arrays
    gathered  the contrast side runs over every global anchor, from the state gathered from all workers
    raw       the worker normalises its own raw fp32 encoder rows into its slice of the global batch first, and the
              gradients are with respect to the raw rows
    update    "" no temperature update, "fused" with the step, "after" as a call of its own behind it
"""
import torch

from paper_2407_01445_amd import binding as fc

DEVICE = "cuda"


def _case(name, dtype, version, B, b, off, d, N, *, ld=None, records=False, gathered=False, raw=False, update="",
          gamma=0.8, eps=1e-14, rho=8.5, noise=0.5):
    c = dict(dtype=dtype, version=version, B=B, b=b, off=off, d=d, ld=d if ld is None else ld, N=N, records=records,
             gathered=gathered, raw=raw, update=update, gamma=gamma, eps=eps, rho=rho, noise=noise)
    return dict(c, name=name) if name else c


def listed():
    return [
        # fp32 embeddings: the smallest whole batch (a check against another implementation, a toy run)
        _case("f32_64_d32", "f32", 1, 64, 64, 0, 32, 1024, rho=0.0),
        # fp32 embeddings at 128 anchors per worker on 8 workers, the medium setting of the method's own runs
        _case("f32_128_of_1024_d512", "f32", 3, 1024, 128, 384, 512, 2_700_000, gamma=0.6, rho=6.5),
        # fp32 embeddings, the whole batch on one worker, one temperature per sample and their update with the step
        _case("f32_1024_d512_v2", "f32", 2, 1024, 1024, 0, 512, 2_700_000, update="fused"),
        # the medium setting in bf16: the smallest step a training run makes, all latency
        _case("bf16_128_of_1024_d512", "bf16", 3, 1024, 128, 384, 512, 2_700_000, gamma=0.6, rho=6.5),
        # one worker holding a small batch
        _case("bf16_1024_d512", "bf16", 3, 1024, 1024, 0, 512, 2_700_000, rho=6.5),
        # few anchors against a batch of many workers
        _case("bf16_256_of_8192_d512", "bf16", 3, 8192, 256, 1280, 512, 9_100_000, gamma=0.6),
        # a worker's whole iteration around its encoders: raw rows in, gradients of raw rows out, one temperature per
        # sample, stepped behind the step from records
        _case("bf16_256_of_2048_d512_raw", "bf16", 2, 2048, 256, 768, 512, 9_100_000, records=True, raw=True,
              update="after"),
        # the largest setting of the method's own runs (640 anchors per worker) with the contrast side complete
        _case("bf16_640_of_5120_d512_gathered", "bf16", 3, 5120, 640, 3200, 512, 9_100_000, gathered=True, gamma=0.6,
              eps=1e-6),
        # a batch that is no multiple of anything, rows padded
        _case("bf16_1000_of_4000_d760_ragged", "bf16", 0, 4000, 1000, 2000, 760, 2_700_000, ld=768, gamma=0.6),
        # one worker holding a large batch
        _case("bf16_4096_d768_v2", "bf16", 2, 4096, 4096, 0, 768, 9_100_000),
        # the large workload: 1024 anchors of 32 workers' batch, per-sample temperatures stepped with the step
        _case("bf16_1024_of_32768_d1024_v2", "bf16", 2, 32768, 1024, 17408, 1024, 315_000_000, records=True,
              update="fused", gamma=0.6, eps=1e-6, noise=0.3),
        # the same with the contrast side over all 32768 anchors
        _case("bf16_1024_of_32768_d1024_v2_gathered", "bf16", 2, 32768, 1024, 17408, 1024, 9_100_000, records=True,
              gathered=True, gamma=0.6, eps=1e-6, noise=0.3),
    ]


def draw(rng):
    """Another step of the same ranges: 32 .. 4096 anchors per worker on 1 .. 32 workers, widths 64 .. 1024."""
    while True:
        f32 = rng.random() < 0.25
        lo, hi = (32, 1024) if f32 else (64, 4096)
        b = int(round(lo * (hi / lo) ** rng.random()))
        shape = rng.random()
        if shape < 0.5:                                   # whole tiles, as most users pick them
            b = max(lo, b // 64 * 64)
        elif shape < 0.8:
            b = max(lo, b // 8 * 8)
        workers = rng.choice([1, 1, 2, 4, 8, 8, 16, 32])
        B = b * workers
        d = rng.choice([64, 128, 256, 384, 512, 512, 640, 768, 1024]) if rng.random() < 0.6 else 8 * rng.randint(8, 128)
        if B > 32768 or b * B * d > (1024 * 5120 * 512 // 5 if f32 else 1024 * 32768 * 1024):
            continue
        version = rng.choice([0, 1, 2, 3, 3])
        gathered = workers > 1 and rng.random() < 0.3
        update = "" if version == 1 else rng.choice(["", "", "fused", "after"])
        return _case(None, "f32" if f32 else "bf16", version, B, b, rng.randrange(workers) * b, d,
                     rng.choice([2_700_000, 9_100_000]), ld=d + rng.choice([0, 0, 0, 8, 64]),
                     records=version == 2 and rng.random() < 0.5, gathered=gathered, raw=rng.random() < 0.25, update=update,
                     gamma=rng.choice([0.2, 0.6, 0.8, 1.0]), eps=rng.choice([1e-14, 1e-6]), rho=rng.choice([6.5, 8.5]))


def _unit(x):
    return x / x.norm(dim=1, keepdim=True)


def _distinct(n, N, gen):
    """n distinct indices from [0, N) in random order."""
    got = torch.empty(0, dtype=torch.int64, device=DEVICE)
    while got.numel() < n:
        more = torch.randint(0, N, (2 * n,), generator=gen, device=DEVICE)
        got = torch.unique(torch.cat([got, more]))
    return got[torch.randperm(got.numel(), generator=gen, device=DEVICE)[:n]].contiguous()


def _visited(n, gen):
    """Moving averages of a run under way: spread over two orders of magnitude around 0.3."""
    return torch.exp(torch.randn(n, generator=gen, device=DEVICE) - 1.2)


class _State:
    pass


def prepare(case, seed):
    """Inputs, state and the handles a training loop keeps (config, buffers, workspace)."""
    c = case
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    B, b, off, d, ld, N, v2 = c["B"], c["b"], c["off"], c["d"], c["ld"], c["N"], c["version"] == 2
    store = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    f32 = dict(dtype=torch.float32, device=DEVICE)
    s = _State()
    s.case = c
    image = _unit(torch.randn(B, d, generator=gen, **f32))
    text = _unit(image + c["noise"] * torch.randn(B, d, generator=gen, **f32))
    s.img, s.txt = torch.zeros(B, ld, dtype=store, device=DEVICE), torch.zeros(B, ld, dtype=store, device=DEVICE)
    s.img[:, :d], s.txt[:, :d] = image, text
    if c["raw"]:          # encoder outputs of very different length
        length = torch.exp(0.5 * torch.randn(2, b, 1, generator=gen, **f32) + 2.0)
        s.raw_img = (image[off:off + b] * length[0]).contiguous()
        s.raw_txt = (text[off:off + b] * length[1]).contiguous()
        s.norm_img, s.norm_txt = torch.empty(b, **f32), torch.empty(b, **f32)
    del image, text
    s.idx = _distinct(b, N, gen)
    # per-sample state; one sample in eight has not been visited yet
    fields = ["u_img", "tau_img", "m_img", "v_img", "u_txt", "tau_txt", "m_txt", "v_txt"]
    if c["records"]:
        s.records = torch.zeros(N, 8, **f32)
        columns = {n: s.records[:, i] for i, n in enumerate(fields)}
    else:
        columns = {n: torch.zeros(N, **f32) for n in (fields if v2 else ["u_img", "u_txt"])}
    for side in ("img", "txt"):
        u = columns["u_" + side]
        u.copy_(_visited(N, gen))
        u[torch.randint(0, 8, (N,), generator=gen, device=DEVICE, dtype=torch.int8) == 0] = 0.0
        if v2:
            columns["tau_" + side].uniform_(0.05, 0.09, generator=gen)
    s.u_img, s.u_txt = columns["u_img"], columns["u_txt"]
    s.tau = None if v2 else torch.full((1,), 0.07, **f32)
    s.d_img, s.d_txt = torch.empty(b, d, **f32), torch.empty(b, d, **f32)
    s.loss = torch.empty(1, **f32)
    s.d_tau = torch.empty(1, **f32) if c["version"] in (0, 3) else None
    s.d_tau_img, s.d_tau_txt = (torch.empty(b, **f32), torch.empty(b, **f32)) if v2 else (None, None)
    # what a worker sends to the others; a worker that holds the whole batch has nobody to send it to
    s.u_new_img, s.u_new_txt = (torch.empty(b, **f32), torch.empty(b, **f32)) if b < B else (None, None)
    more = {}
    if c["gathered"]:
        more = dict(u_glob_img=_visited(B, gen), u_glob_txt=_visited(B, gen))
        if v2:
            more["tau_glob_img"] = torch.empty(B, **f32).uniform_(0.05, 0.09, generator=gen)
            more["tau_glob_txt"] = torch.empty(B, **f32).uniform_(0.05, 0.09, generator=gen)
    if c["raw"]:
        more.update(norm_img=s.norm_img, norm_txt=s.norm_txt)
    stride = 8 if c["records"] else 1
    s.cfg = fc.make_config(version=c["version"], emb_dtype=fc.BF16 if c["dtype"] == "bf16" else fc.F32, B=B, b=b, off=off,
                           d=d, N=N, gamma=c["gamma"], eps=c["eps"], rho=c["rho"], ld_img=ld, ld_txt=ld,
                           flags=fc.GATHERED_STATE if c["gathered"] else 0, state_stride=stride)
    tau = dict(tau_img=columns["tau_img"], tau_txt=columns["tau_txt"]) if v2 else dict(tau=s.tau)
    s.bufs = fc.make_buffers(img_glob=s.img, txt_glob=s.txt, idx=s.idx, u_img=s.u_img, u_txt=s.u_txt, d_img=s.d_img,
                             d_txt=s.d_txt, loss=s.loss, d_tau=s.d_tau, d_tau_img=s.d_tau_img, d_tau_txt=s.d_tau_txt,
                             u_new_img=s.u_new_img, u_new_txt=s.u_new_txt, **tau, **more)
    s.workspace = torch.empty(fc.fastclip_workspace_bytes(s.cfg), dtype=torch.uint8, device=DEVICE)
    s.tau_state = None
    if c["update"]:
        s.upd = fc.make_tau_update(optimizer=fc.TAU_ADAMW, step=100, lr=1e-4, beta1=0.9, beta2=0.999, tau_min=0.03,
                                   state_stride=stride)
        moments = ({n: columns[n] for n in ("m_img", "v_img", "m_txt", "v_txt")} if v2
                   else dict(m=torch.zeros(1, **f32), v=torch.zeros(1, **f32)))
        s.tau_state = fc.make_tau_state(**tau, **moments)
        s.moments = moments
    # what the step returns: gradients, loss, temperature gradients, and the state it has updated
    s.out = dict(d_img=s.d_img, d_txt=s.d_txt, loss=s.loss, d_tau=s.d_tau, d_tau_img=s.d_tau_img, d_tau_txt=s.d_tau_txt,
                 u_new_img=s.u_new_img, u_new_txt=s.u_new_txt)
    if c["records"]:
        s.out.update(records=s.records)
    else:
        s.out.update(u_img=s.u_img, u_txt=s.u_txt)
        if c["update"]:
            s.out.update(tau, **moments)
    if c["raw"]:
        s.out.update(norm_img=s.norm_img, norm_txt=s.norm_txt)
        size = s.img.element_size()
        s.unit_img = s.img.data_ptr() + off * ld * size      # the worker's slice of the global batch
        s.unit_txt = s.txt.data_ptr() + off * ld * size
    s.out = {k: v for k, v in s.out.items() if v is not None}
    return s


def run(s):
    """One iteration of a worker: the step and what its case puts around it."""
    c = s.case
    if c["raw"]:
        unit = s.cfg.emb_dtype
        fc.fastclip_normalize_rows(s.raw_img, fc.F32, c["d"], c["b"], c["d"], s.unit_img, unit, c["ld"], s.norm_img)
        fc.fastclip_normalize_rows(s.raw_txt, fc.F32, c["d"], c["b"], c["d"], s.unit_txt, unit, c["ld"], s.norm_txt)
    if c["update"] == "fused":
        fc.fastclip_step_update_tau(s.cfg, s.bufs, s.upd, s.tau_state, s.workspace)
    else:
        fc.fastclip_step(s.cfg, s.bufs, s.workspace)
        if c["update"] == "after":
            fc.fastclip_temperature_update(c["version"], s.upd, s.tau_state, s.idx, c["b"], c["N"], s.d_tau, s.d_tau_img,
                                           s.d_tau_txt)
    return s.out


def work(case):
    """Every embedding, output and touched state word once; the similarities once where both strips are the same
    products (the whole batch local), else twice; one contraction per side."""
    c = case
    B, b, d = c["B"], c["b"], c["d"]
    size = 2 if c["dtype"] == "bf16" else 4
    per_sample = 2 * (1 + (1 if c["version"] == 2 else 0) + (2 if c["version"] == 2 and c["update"] else 0))
    written = 2 * (1 + (3 if c["version"] == 2 and c["update"] else 0))
    moved = 2 * B * d * size + 2 * b * d * 4 + b * (8 + 4 * per_sample + 4 * written)
    if c["gathered"]:
        moved += B * 4 * (4 if c["version"] == 2 else 2)
    if c["raw"]:
        moved += 2 * b * d * 4
    return {"bytes": moved, "flops": (3 if b == B else 4) * 2.0 * b * B * d}


def tolerance(case):
    """Four times what a float64 evaluation of the same step differs by, at worst over these ranges.  fp32: dot products
    and sums are carried in fp64, the rounding of stored exponentials, coefficients and outputs is left (9e-8, 4e-7).
    bf16: the exponentials are rounded to 8 bits as operands of the gradient contractions, which averages out over the
    batch (5e-4 and 8e-3 at 100 pairs, 1e-5 at 10,000)."""
    return {"rel": 1e-6, "max": 4e-6} if case["dtype"] == "f32" else {"rel": 2e-3, "max": 3.2e-2}
