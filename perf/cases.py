"""The work a training program has this framework do, as cases a measuring program can run.

A case is one clipped optimizer step, one gradient norm or one layer-streamed step,
through the public entry points of ``paper_2608_11919_amd``, on the state a program
keeps between steps.  The parameter lists are decoder models (the repository's
benchmark shapes and generic smaller ones), low-rank adapter sets and lists of odd
sizes.  ``exact`` restates the arithmetic in 64 bits with torch alone.

Tensors that a case owns are views into flat buffers, each starting at a multiple of
512 elements (torch's own allocations start at multiples of 512 bytes), so that the
outputs are a handful of buffers however many tensors the list has.
"""
import math
import random

import torch

import paper_2608_11919_amd as lt

LR, BETA1, BETA2, EPS, WEIGHT_DECAY = 1e-4, 0.9, 0.999, 1e-8, 0.01
MAX_NORM = 1.0
STEP = 100            # the step being applied: a run that is under way
PITCH = 512           # elements between the starts of two tensors, at least
POWER_BLOCKS = (64, 128, 256, 512, 1024, 2048, 4096, 8192)
OTHER_BLOCKS = (192, 320, 576, 768, 1536, 3072, 5120, 12288, 16384, 65536)


# ---------------------------------------------------------------------- cases

def listed():
    return [
        # The benchmark's tiny set, four fp32-gradient tensors of 2.6M parameters in
        # all: a step whose launches and latencies outweigh its bytes.
        dict(name="tiny_set", path="step8", kind="tiny", block=256, map="linear", grad="f32",
             copy=False),
        # Low-rank adapters on the four attention projections of a 36-layer model
        # (rank 16): 288 small tensors, 9.4M parameters, 8-bit states in small blocks.
        dict(name="adapters", path="step8", kind="adapters", layers=36, hidden=2048, rank=16,
             block=512, map="dynamic", grad="bf16", copy=False),
        # 240 tensors of odd sizes from one element to half a million (biases, norms,
        # convolutions, odd vocabularies): partial blocks and granules everywhere.
        dict(name="odd_sizes", path="step8", kind="odd", count=240, largest=500000, sizes=7,
             block=1024, map="linear", grad="bf16", copy=True),
        # One decoder layer of the 3B-class model through the optimizer object with
        # its defaults (block 4096, dynamic codes): the call a training loop makes.
        dict(name="layer_optimizer", path="opt", kind="decoder", layers=1, hidden=2048, ffn=11008,
             kv=256, vocab=0, block=4096, map="dynamic", grad="bf16", copy=False, slice=0.0),
        # The hybrid operator on one layer of the 27B-class model: 8-bit states for 2%
        # of the parameters, fp32 states for the rest, and the bf16 weight copy.
        dict(name="hybrid_optimizer", path="opt", kind="decoder", layers=1, hidden=5120,
             ffn=17408, kv=1024, vocab=0, block=4096, map="dynamic", grad="bf16", copy=True,
             slice=0.02),
        # The headline workload: embedding and 36 layers, 325 tensors, 3.09e9 parameters.
        dict(name="full_model", path="step8", kind="decoder", layers=36, hidden=2048, ffn=11008,
             kv=256, vocab=151936, block=2048, map="linear", grad="bf16", copy=False),
        # The paper's block size with the dynamic codes and the bf16 copy for the next
        # forward pass, on six layers of the 3B-class model.
        dict(name="paper_block", path="step8", kind="decoder", layers=6, hidden=2048, ffn=11008,
             kv=256, vocab=0, block=4096, map="dynamic", grad="bf16", copy=True),
        # A block size that is no power of two (whole rows of a hidden size of 768) on a
        # small 12-layer decoder with its embedding, fp32 gradients.
        dict(name="row_blocks", path="step8", kind="decoder", layers=12, hidden=768, ffn=3072,
             kv=768, vocab=32000, block=768, map="linear", grad="f32", copy=False),
        # fp32 states on the same small decoder: the part of the hybrid operator that
        # keeps full-precision moments, called on its own.
        dict(name="fp32_states", path="step32", kind="decoder", layers=12, hidden=768, ffn=3072,
             kv=768, vocab=32000, grad="f32", copy=False),
        # The norm summed as a backward pass delivers the gradients, layer by layer.
        dict(name="norm_on_arrival", path="arrival", kind="decoder", layers=12, hidden=2048,
             ffn=11008, kv=256, vocab=0, grad="bf16"),
        # Norm and clip coefficient of fp32 gradients without a workspace, as code under
        # capture calls it.
        dict(name="norm_noalloc", path="norm", kind="decoder", layers=4, hidden=2048, ffn=11008,
             kv=256, vocab=0, grad="f32"),
        # Weights, gradients and 8-bit states in pinned host memory, streamed through
        # the GPU layer by layer with the gradients kept in HBM between the passes.
        dict(name="streamed", path="streamed", kind="decoder", layers=8, hidden=1024, ffn=4096,
             kv=256, vocab=0, block=4096, map="dynamic", grad="bf16", copy=False, keep=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed kinds, over their whole ranges."""
    path = rng.choice(["step8", "step8", "step8", "opt", "opt", "step32", "arrival", "norm",
                       "streamed"])
    c = dict(path=path, grad=rng.choice(["bf16", "bf16", "f32"]))
    if path in ("step8", "step32", "norm"):
        kind = rng.choice(["adapters", "odd", "decoder", "decoder"])
    else:
        kind = "decoder"
    c["kind"] = kind
    if kind == "adapters":
        c.update(layers=rng.randint(4, 48), hidden=64 * rng.randint(8, 80),
                 rank=rng.choice([4, 8, 16, 32, 64]))
    elif kind == "odd":
        c.update(count=_log_int(rng, 8, 400), largest=_log_int(rng, 1000, 2000000),
                 sizes=rng.randrange(1 << 20))
    else:
        hidden = 64 * _log_int(rng, 4, 40)
        layers = 1 if path == "opt" else rng.randint(1, 4) if path == "streamed" else \
            rng.randint(1, 16)
        if path == "opt":
            hidden = 64 * _log_int(rng, 8, 80)
        c.update(layers=layers, hidden=hidden, ffn=hidden * rng.randint(10, 20) // 4 | 1,
                 kv=64 * rng.randint(1, max(1, hidden // 64)),
                 vocab=0 if path in ("opt", "streamed", "arrival") else
                 rng.choice([0, _log_int(rng, 1000, 60000)]))
    if path in ("step8", "opt", "streamed"):
        c.update(block=rng.choice(POWER_BLOCKS if rng.random() < 0.7 else OTHER_BLOCKS),
                 map=rng.choice(["linear", "dynamic"]), copy=rng.random() < 0.3)
    if path == "step32":
        c["copy"] = rng.random() < 0.3
    if path == "opt":
        c["slice"] = rng.choice([0.0, 0.0, 0.02, 0.2])
    if path == "streamed":
        c["keep"] = rng.random() < 0.7
    return c


# ---------------------------------------------------------------------- sizes

def _layer(h, ffn, kv):
    """q, k, v, o, gate, up, down and the two norms of one decoder layer."""
    return [h * h, kv * h, kv * h, h * h, ffn * h, ffn * h, h * ffn, h, h]


def _numels(case):
    kind = case["kind"]
    if kind == "tiny":
        return [512 * 1024, 1024 * 1024, 2048 * 512, 1024]
    if kind == "adapters":
        return case["layers"] * 4 * [case["rank"] * case["hidden"]] * 2
    if kind == "odd":
        r = random.Random(case["sizes"])
        return [1, case["largest"] | 1] + [_log_int(r, 1, case["largest"])
                                           for _ in range(case["count"] - 2)]
    layer = _layer(case["hidden"], case["ffn"], case["kv"])
    return ([case["vocab"] * case["hidden"]] if case["vocab"] else []) + case["layers"] * layer


class _Flat:
    """One tensor per size, as views of one flat buffer (zeros between them)."""

    def __init__(self, sizes, dtype, pitch=PITCH, pinned=False):
        at = [0]
        for n in sizes:
            at.append(at[-1] + -(-max(n, 1) // pitch) * pitch)
        self.flat = torch.zeros(at[-1], dtype=dtype, pin_memory=True) if pinned else \
            torch.zeros(at[-1], dtype=dtype, device="cuda")
        self.views = [self.flat[a:a + n] for a, n in zip(at, sizes)]


# --------------------------------------------------------------------- values

def _decades(bits):
    """Magnitudes of the dynamic codes of `bits` magnitude bits, in 64 bits."""
    out = [0.0]
    for c in range(1, 1 << bits):
        p = c.bit_length() - 1
        f = c - (1 << p)
        out.append((0.1 + 0.9 * ((f + 1) / (1 << p))) * 10.0 ** -(bits - 1 - p))
    return torch.tensor(out, dtype=torch.float64, device="cuda")


def _blocks(x, B):
    """x as rows of one block each, zeros after its end."""
    nb = -(-x.numel() // B)
    if nb * B != x.numel():
        x = torch.cat([x, x.new_zeros(nb * B - x.numel())])
    return x.view(nb, B)


def _quantize(x, B, dynamic, signed, tables):
    """Codes and block scales of a moment, as earlier steps would have left them."""
    rows = _blocks(x, B)
    amax = rows.abs().amax(1)
    a = rows / amax.clamp_min(1e-30).unsqueeze(1)
    if dynamic:
        mids = tables[signed]
        q = torch.bucketize(a.abs(), mids).to(torch.uint8)
        if signed:
            q = torch.where(a < 0, q | 0x80, q).view(torch.int8)
    else:
        q = torch.round(a * 127).to(torch.int8) if signed else torch.round(a * 255).to(torch.uint8)
    return q.reshape(-1)[:x.numel()], amax


def _gradient(n, gen):
    """Heavy-tailed values (Student's t with three degrees of freedom) around 1e-3."""
    r = lambda: torch.randn(n, device="cuda", generator=gen)
    chi = r().square_()
    chi.add_(r().square_()).add_(r().square_())
    return r().mul_(1e-3).div_(chi.div_(3.0).sqrt_().clamp_min_(0.02))


def _inputs(case, seed, pinned=False):
    """Weights, gradients and moments of the case's list, from the seed alone: a dict of
    _Flat buffers (codes and scales, or fp32 moments, or none for the norms)."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed * 1000003 + 17)
    sizes = _numels(case)
    gdt = torch.bfloat16 if case["grad"] == "bf16" else torch.float32
    x = {"numels": sizes, "g": _Flat(sizes, gdt, pinned=pinned)}
    path = case["path"]
    bits8 = path in ("step8", "streamed", "opt")
    states32 = path == "step32" or case.get("slice", 0.0) > 0.0
    if path in ("norm", "arrival"):
        for g in x["g"].views:
            g.copy_(_gradient(g.numel(), gen))
        return x
    x["w"] = _Flat(sizes, torch.float32, pinned=pinned)
    if states32:
        x["m"], x["v"] = _Flat(sizes, torch.float32), _Flat(sizes, torch.float32)
    if bits8:
        B, dynamic = case["block"], case["map"] == "dynamic"
        nb = [-(-n // B) for n in sizes]
        x["mq"] = _Flat(sizes, torch.int8, pinned=pinned)
        x["vq"] = _Flat(sizes, torch.uint8, pinned=pinned)
        x["ma"] = _Flat(nb, torch.float32, 128, pinned=pinned)
        x["va"] = _Flat(nb, torch.float32, 128, pinned=pinned)
        tables = None
        if dynamic:
            mid = lambda t: ((t[1:] + t[:-1]) * 0.5).float()
            tables = {True: mid(_decades(7)), False: mid(_decades(8))}
    for k, n in enumerate(sizes):
        x["w"].views[k].copy_(torch.randn(n, device="cuda", generator=gen).mul_(0.02))
        x["g"].views[k].copy_(_gradient(n, gen))
        m = torch.randn(n, device="cuda", generator=gen).mul_(3e-4)
        v = torch.randn(n, device="cuda", generator=gen).square_().add_(0.05).mul_(1e-6)
        if states32:
            x["m"].views[k].copy_(m)
            x["v"].views[k].copy_(v)
        if bits8:
            for q, a, t, signed in (("mq", "ma", m, True), ("vq", "va", v, False)):
                codes, scales = _quantize(t, B, dynamic, signed, tables)
                x[q].views[k].copy_(codes)
                x[a].views[k].copy_(scales)
    return x


def _scalars():
    z = lambda dt: torch.zeros(1, dtype=dt, device="cuda")
    return {"sq_total": z(torch.float64), "status": z(torch.int32), "coef": z(torch.float32),
            "total_norm": z(torch.float32)}


def _map(case):
    return lt.LT_MAP_DYNAMIC if case["map"] == "dynamic" else lt.LT_MAP_LINEAR


# ------------------------------------------------------------- prepare and run

def prepare(case, seed):
    path, sizes = case["path"], _numels(case)
    x = _inputs(case, seed, pinned=path == "streamed")
    s = {"case": case, "x": x, **_scalars()}
    K = len(sizes)
    space = lambda n: torch.empty(max(n, 256), dtype=torch.uint8, device="cuda")
    if path in ("step8", "step32"):
        s["ws_norm"] = space(lt.lt_grad_sqnorm_workspace_bytes(sizes))
        s["ws_step"] = space(lt.lt_step_workspace_bytes(K) if path == "step8" else
                             lt.lt_adamw_fp32_workspace_bytes(K))
        if case["copy"]:
            x["wb"] = _Flat(sizes, torch.bfloat16)
    elif path == "opt":
        opt = lt.Hybrid8bitAdamW(x["w"].views, lr=LR, betas=(BETA1, BETA2), eps=EPS,
                                 weight_decay=WEIGHT_DECAY, max_norm=MAX_NORM,
                                 block_size=case["block"], slice_fraction=case["slice"] or None,
                                 bf16_copy=case["copy"], code_map=_map(case))
        pick = lambda key, idx: [x[key].views[i] for i in idx] if idx else []
        opt.load_state_dict({
            "step_count": STEP - 1, "consecutive_skips": 0, "is_8bit": list(opt.is_8bit),
            "hyper": dict(lr=LR, betas=(BETA1, BETA2), eps=EPS, weight_decay=WEIGHT_DECAY,
                          max_norm=MAX_NORM, block_size=case["block"], code_map=_map(case)),
            "m_codes": pick("mq", opt.idx8), "m_absmax": pick("ma", opt.idx8),
            "v_codes": pick("vq", opt.idx8), "v_absmax": pick("va", opt.idx8),
            "exp_avg": pick("m", opt.idx32), "exp_avg_sq": pick("v", opt.idx32)})
        s["opt"] = opt
    elif path == "arrival":
        s["acc"] = lt.GradNormAccumulator(sizes, "cuda")
        s["sq"] = torch.zeros(K, dtype=torch.float64, device="cuda")
    elif path == "norm":
        s["sq"] = torch.zeros(K, dtype=torch.float64, device="cuda")
    elif path == "streamed":
        s["first"] = list(range(0, K + 1, 9))
        gdt = lt.LT_DTYPE_BF16 if case["grad"] == "bf16" else lt.LT_DTYPE_F32
        s["ws"] = space(lt.lt_streamed_workspace_bytes(sizes, s["first"], gdt, case["block"], 3,
                                                       case["copy"], case["keep"]))
        s["streams"] = [torch.cuda.Stream() for _ in range(3)]
        if case["copy"]:
            x["wb"] = _Flat(sizes, torch.bfloat16, pinned=True)
    torch.cuda.synchronize()
    return s


def run(s):
    case, x = s["case"], s["x"]
    path = case["path"]
    hyper = dict(lr=LR, beta1=BETA1, beta2=BETA2, eps=EPS, weight_decay=WEIGHT_DECAY, step=STEP)
    norm = {k: s[k] for k in ("sq_total", "total_norm", "coef", "status")}
    if path in ("step8", "step32"):
        g = x["g"].views
        lt.lt_grad_sqnorm(g, s["sq_total"], s["status"], workspace=s["ws_norm"])
        lt.lt_clip_coef(s["sq_total"], MAX_NORM, s["coef"], s["total_norm"])
        copies = x["wb"].views if case["copy"] else None
        if path == "step8":
            lt.lt_hybrid8bit_adamw_step(x["w"].views, g, x["mq"].views, x["ma"].views,
                                        x["vq"].views, x["va"].views, case["block"],
                                        coef=s["coef"], status=s["status"],
                                        workspace=s["ws_step"], params_bf16=copies,
                                        code_map=_map(case), **hyper)
            keys = ("w", "mq", "ma", "vq", "va")
        else:
            lt.lt_adamw_fp32_step(x["w"].views, g, x["m"].views, x["v"].views, coef=s["coef"],
                                  status=s["status"], workspace=s["ws_step"],
                                  params_bf16=copies, **hyper)
            keys = ("w", "m", "v")
        return {**norm, **{k: x[k].flat for k in keys + (("wb",) if case["copy"] else ())}}
    if path == "opt":
        opt = s["opt"]
        opt.step(x["g"].views)
        return {"total_norm": opt.total_norm, "w": x["w"].flat, "mq": opt.m_codes,
                "ma": opt.m_absmax, "vq": opt.v_codes, "va": opt.v_absmax, "m": opt.exp_avg,
                "v": opt.exp_avg_sq, **({"wb": opt.params_bf16} if case["copy"] else {})}
    if path in ("arrival", "norm"):
        g = x["g"].views
        if path == "arrival":
            for first in range(len(g) - 9, -1, -9):
                s["acc"].add(first, g[first:first + 9])
            s["acc"].finish(s["sq_total"], s["status"], s["sq"])
        else:
            lt.lt_grad_sqnorm_noalloc(g, s["sq_total"], s["status"], s["sq"])
        lt.lt_clip_coef(s["sq_total"], MAX_NORM, s["coef"], s["total_norm"])
        return {**norm, "sq": s["sq"]}
    copies = x["wb"].views if case["copy"] else None
    cs, hs, ds = s["streams"]
    lt.lt_streamed_hybrid8bit_adamw_step(
        x["w"].views, x["g"].views, x["mq"].views, x["ma"].views, x["vq"].views, x["va"].views,
        s["first"], case["block"], max_norm=MAX_NORM, ring_slots=3, sq_total=s["sq_total"],
        coef=s["coef"], status=s["status"], total_norm=s["total_norm"], workspace=s["ws"],
        compute_stream=cs, h2d_stream=hs, d2h_stream=ds, params_bf16=copies,
        code_map=_map(case), keep_grads=case["keep"], **hyper)
    lt.lt_read_status(s["status"], cs)  # the host state is read next: wait for it
    return {**norm, **{k: x[k].flat for k in ("w", "mq", "ma", "vq", "va") +
                       (("wb",) if case["copy"] else ())}}


# ----------------------------------------------------------- work and tolerance

def work(case):
    """Each gradient, weight and state read once, each weight, state and copy written
    once; two operations per element for the norm, about twenty for the update."""
    sizes = _numels(case)
    n = sum(sizes)
    g = 2 if case["grad"] == "bf16" else 4
    path = case["path"]
    if path in ("norm", "arrival"):
        return {"bytes": n * g + 8 * len(sizes), "flops": 2 * n}
    states = 16
    if path in ("step8", "streamed") or (path == "opt" and not case["slice"]):
        states = 4 + 16 / case["block"]
    elif path == "opt":
        states = 16 - (12 - 16 / case["block"]) * case["slice"]
    return {"bytes": n * (g + 8 + states + (2 if case["copy"] else 0)), "flops": 22 * n}


def tolerance(case):
    """The order of the norm's sum and of every operation of the update is part of the
    interface (include/lazytrain.h), so every result is the same bits."""
    return "exact"


# ------------------------------------------------------------------------ exact

def exact(case, seed):
    """The step in 64 bits from the same inputs; codes, being roundings, have no such value."""
    x = _inputs(case, seed)
    sizes, path = x["numels"], case["path"]
    sq = torch.stack([g.double().square().sum() for g in x["g"].views])
    S = sq.sum().reshape(1)
    norm = S.sqrt()
    coef = torch.clamp(MAX_NORM / (norm + 1e-6), max=1.0)
    out = {"sq_total": S, "total_norm": norm, "coef": coef, "status": None}
    if path in ("norm", "arrival"):
        return {**out, "sq": sq}
    bits8 = [path in ("step8", "streamed") or (path == "opt" and not case["slice"])] * len(sizes)
    if path == "opt" and case["slice"]:
        total, taken = sum(sizes), 0  # largest first, while the sum stays within the fraction
        for k in sorted(range(len(sizes)), key=lambda i: (-sizes[i], i)):
            if taken + sizes[k] <= case["slice"] * total:
                bits8[k] = True
                taken += sizes[k]
    if any(bits8):
        dynamic = case["map"] == "dynamic"
        B = case["block"]
        if dynamic:
            t7, t8 = _decades(7), _decades(8)
            m_of = torch.cat([t7, -t7])
        nb = [-(-n // B) for n in sizes]
    got = {"w": _Flat(sizes, torch.float64)}
    lists = {"m": [], "v": [], "ma": [], "va": []}
    for k, n in enumerate(sizes):
        if bits8[k]:
            mq, vq = x["mq"].views[k], x["vq"].views[k]
            scale = lambda a: a.double().repeat_interleave(B)[:n]
            if dynamic:
                m = m_of[mq.view(torch.uint8).int()] * scale(x["ma"].views[k])
                v = t8[vq.int()] * scale(x["va"].views[k])
            else:
                m = mq.double() * scale(x["ma"].views[k]) / 127
                v = vq.double() * scale(x["va"].views[k]) / 255
        else:
            m, v = x["m"].views[k].double(), x["v"].views[k].double()
        g = x["g"].views[k].double() * coef
        m = BETA1 * m + (1 - BETA1) * g
        v = BETA2 * v + (1 - BETA2) * g.square()
        den = v.sqrt() / math.sqrt(1 - BETA2 ** STEP) + EPS
        got["w"].views[k].copy_(x["w"].views[k].double() * (1 - LR * WEIGHT_DECAY) -
                                LR / (1 - BETA1 ** STEP) * m / den)
        if bits8[k]:
            lists["ma"].append(_blocks(m.abs(), B).amax(1))
            lists["va"].append(_blocks(v, B).amax(1))
        else:
            lists["m"].append(m)
            lists["v"].append(v)
        del g, den
    w = got["w"].flat
    if path == "opt":
        return {"total_norm": norm, "w": w, "mq": None, "vq": None, **lists,
                **({"wb": got["w"].views} if case["copy"] else {})}

    def flat(key, counts, pitch):
        f = _Flat(counts, torch.float64, pitch)
        for a, b in zip(f.views, lists[key]):
            a.copy_(b)
        return f.flat

    out["w"] = w
    if path == "step32":
        out.update(m=flat("m", sizes, PITCH), v=flat("v", sizes, PITCH))
    else:
        out.update(mq=None, vq=None, ma=flat("ma", nb, 128), va=flat("va", nb, 128))
    if case["copy"]:
        out["wb"] = w
    return out
