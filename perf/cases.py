"""The calls whose time is measured: what a program that uses this library has it do, through `binding.FastWavenet`.

A case names a model (layer kind, operand type, channels, layers, dilation pattern, filter width), a batch of
streams and one way to call the model:

  generate   a new generation: observe a prefix step by step (its logits come back), then draw samples
  steps      a latency-bound loop: one observed step per call, one call after the other
  online     online prediction: one call that runs `steps` observed steps on the step kernels
  teacher    teacher forcing of whole sequences, time-parallel (scoring a batch of recordings)
  prime      a long prefix primes the queues time-parallel, then a few observed steps continue from it

Generated classes feed back into the model, so two correct implementations that round differently part ways for
good once one draw falls on the other side of a CDF boundary.  In float32 that is rare over a short stretch; in
bf16 it is not, so bf16 models are measured through the calls that return logits of observed samples (the same
step kernels).
"""
import math

import torch

import workloads as W
from paper_1611_09482_amd import binding

KINDS = {"relu": W.RELU, "relu_residual": W.RELU_RESIDUAL, "gated": W.GATED}
DTYPES = {"f32": W.F32, "bf16": W.BF16}


def _case(name, call, kind, dtype, channels, layers, per_block, batch, steps, skip=0, head=0, rate=2, width=2,
          prefix=0):
    c = {"call": call, "kind": kind, "dtype": dtype, "channels": channels, "skip": skip, "head": head,
         "layers": layers, "per_block": per_block, "rate": rate, "width": width, "batch": batch, "steps": steps,
         "prefix": prefix}
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest model, one stream: a sample is a chain of dependent operations
        _case("toy_generate_b1", "generate", "relu", "f32", 32, 5, 5, 1, 200, prefix=40),
        # real-time use of a small WaveNet: one call per sample, the launch counts
        _case("r32_single_steps_b1", "steps", "gated", "f32", 32, 20, 10, 1, 24, skip=256, head=256),
        # the same model generating for many listeners at once
        _case("r32_generate_b64", "generate", "gated", "f32", 32, 20, 10, 64, 48, skip=256, head=256, prefix=48),
        # the benchmark model on its full batch
        _case("r64_bf16_online_b256", "online", "gated", "bf16", 64, 30, 10, 256, 200, skip=512, head=512),
        # its two-block variant on a ragged batch
        _case("r64_bf16_online_l20_b100", "online", "gated", "bf16", 64, 20, 10, 100, 120, skip=512, head=512),
        # filter width 3 on the benchmark's layer shape
        _case("r64_bf16_online_w3_b256", "online", "gated", "bf16", 64, 14, 7, 256, 100, skip=512, head=512, rate=3,
              width=3),
        # a wide ReLU + residual decoder
        _case("c512_generate_b32", "generate", "relu_residual", "f32", 512, 25, 5, 32, 32, prefix=16),
        # a gated float32 stack that no specialised kernel was written for
        _case("r64_f32_online_b16", "online", "gated", "f32", 64, 20, 10, 16, 32, skip=256, head=256),
        # scoring recordings with the benchmark model: the largest call
        _case("r64_bf16_teacher_b256", "teacher", "gated", "bf16", 64, 30, 10, 256, 1500, skip=512, head=512),
        # scoring with the small float32 model
        _case("r32_teacher_b64", "teacher", "gated", "f32", 32, 20, 10, 64, 3001, skip=256, head=256),
        # scoring with the wide decoder, sentences of a few hundred symbols
        _case("c512_teacher_b32", "teacher", "relu_residual", "f32", 512, 25, 5, 32, 333),
        # continuing a recording: a long prefix of a few streams, then step by step
        _case("r64_bf16_prime_b4", "prime", "gated", "bf16", 64, 30, 10, 4, 16, skip=512, head=512, prefix=6000),
    ]


def _log(rng, lo, hi):
    """A whole number from lo to hi, spread over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)) - 1e-9)))))


def draw(rng):
    model = rng.choice(("toy", "r32", "r32", "r64_bf16", "r64_bf16", "r64_bf16", "c512", "general"))
    if model == "toy":
        layers = rng.randint(3, 6)
        call = rng.choice(("generate", "steps", "online"))
        return _case("", call, "relu" if rng.random() < 0.5 else "relu_residual", "f32", 32, layers, layers,
                     _log(rng, 1, 64), rng.randint(16, 40), prefix=rng.randint(8, 64) if call == "generate" else 0)
    if model == "r32":
        width = rng.choice((2, 2, 3))
        per = rng.randint(4, 10) if width == 2 else rng.randint(3, 7)
        layers, batch = per * rng.randint(1, 2) + rng.randint(0, 1), _log(rng, 1, 160)
        call = rng.choice(("generate", "steps", "online", "teacher", "prime"))
        steps = {"generate": max(4, min(48, 2000 // batch)), "steps": rng.randint(8, 24), "online": rng.randint(16, 150),
                 "teacher": _log(rng, 16, max(32, 200000 // batch)), "prime": rng.randint(4, 24)}[call]
        prefix = {"generate": rng.randint(8, 64), "prime": _log(rng, 16, max(32, 100000 // batch))}.get(call, 0)
        return _case("", call, "gated", "f32", 32, layers, per, batch, steps, skip=256, head=256,
                     rate=rng.choice((2, width)), width=width, prefix=prefix)
    if model == "r64_bf16":
        width = rng.choice((2, 2, 2, 3))
        per = rng.randint(5, 10) if width == 2 else rng.randint(4, 7)
        layers, batch = per * rng.randint(1, 3) + rng.choice((0, 0, 1)), _log(rng, 1, 400)
        call = rng.choice(("steps", "online", "online", "teacher", "teacher", "prime"))
        steps = {"steps": rng.randint(8, 24), "online": rng.randint(16, 150),
                 "teacher": _log(rng, 16, max(32, 250000 // batch)), "prime": rng.randint(4, 24)}[call]
        prefix = _log(rng, 16, max(32, 100000 // batch)) if call == "prime" else 0
        return _case("", call, "gated", "bf16", 64, layers, per, batch, steps, skip=512, head=512,
                     rate=rng.choice((2, width)), width=width, prefix=prefix)
    if model == "c512":
        per = rng.randint(3, 6)
        layers, batch = per * rng.randint(1, 4) + rng.randint(0, 1), _log(rng, 1, 32)
        call = rng.choice(("generate", "online", "teacher"))
        steps = {"generate": rng.randint(4, 20), "online": rng.randint(4, 48),
                 "teacher": _log(rng, 16, max(32, 10000 // batch))}[call]
        return _case("", call, "relu_residual", "f32", 512, layers, per, batch, steps,
                     prefix=rng.randint(4, 24) if call == "generate" else 0)
    # shapes of the general kernels
    dtype = rng.choice(("f32", "bf16"))
    per = rng.randint(3, 10)
    layers, batch = per * rng.randint(1, 2), _log(rng, 1, 64)
    call = rng.choice(("online", "teacher"))
    steps = rng.randint(8, 32) if call == "online" else _log(rng, 16, max(32, 50000 // batch))
    if rng.random() < 0.5:
        return _case("", call, "gated", dtype, 64, layers, per, batch, steps, skip=rng.choice((128, 256)),
                     head=rng.choice((128, 256)))
    return _case("", call, rng.choice(("relu", "relu_residual")), dtype, rng.choice((64, 128, 256)), layers, per, batch,
                 steps)


def _config(case):
    dil = tuple(case["rate"] ** (i % case["per_block"]) for i in range(case["layers"]))
    return W.ModelConfig(KINDS[case["kind"]], DTYPES[case["dtype"]], case["channels"], dil, case["skip"], case["head"],
                         filter_width=case["width"])


def _weights(case, seed):
    return W.make_weights(_config(case), seed, bias_scale=0.05)


def _recording(batch, length, gen):
    """Observed samples: 8-bit mu-law classes of a few tones in noise, one row per stream."""
    t = torch.arange(length, device="cuda", dtype=torch.float32)
    r = torch.rand((batch, 3, 3), generator=gen, device="cuda")
    tones = (0.25 * r[:, :, :1] * torch.sin(t * (0.01 + 0.3 * r[:, :, 1:2]) + 6.2832 * r[:, :, 2:])).sum(1)
    x = (tones + 0.03 * torch.randn((batch, length), generator=gen, device="cuda")).clamp(-1, 1)
    y = torch.sign(x) * torch.log1p(255 * x.abs()) / math.log(256.0)
    return ((y + 1) * 127.5 + 0.5).to(torch.int32).clamp(0, 255).contiguous()


def _inputs(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7919 * seed + 17)
    drawn = case["call"] == "generate"
    seq = _recording(case["batch"], case["prefix"] if drawn else case["prefix"] + case["steps"], gen)
    u = torch.rand((case["batch"], case["steps"]), generator=gen, device="cuda") if drawn else None
    return seq, u


def prepare(case, seed):
    seq, u = _inputs(case, seed)
    model = binding.from_model(_config(case), _weights(case, seed), max_batch=case["batch"])
    s = {"case": case, "model": model}
    n = case["prefix"]
    if n:
        s["prefix"] = seq[:, :n].contiguous()
    if u is not None:
        s["uniforms"] = u
    elif case["call"] == "steps":
        s["observed"] = [seq[:, i:i + 1].contiguous() for i in range(case["steps"])]
    else:
        s["observed"] = seq[:, n:].contiguous()
    return s


def run(s):
    call, m = s["case"]["call"], s["model"]
    if call == "teacher":
        return m.teacher_forced_parallel(s["observed"])
    m.reset()
    if call == "generate":
        logits = m.step_forced(s["prefix"], check=False)
        return {"logits": logits, "samples": m.generate(s["uniforms"])}
    if call == "steps":
        out = [m.step_forced(x, check=False) for x in s["observed"]]
        m.device_status()
        return out
    if call == "prime":
        return {"prefix": m.prime(s["prefix"], logits=True), "steps": m.step_forced(s["observed"])}
    return m.step_forced(s["observed"])


def work(case):
    cfg, B = _config(case), case["batch"]
    n = case["steps"] + case["prefix"]
    params = cfg.param_count() * (2 if case["dtype"] == "bf16" else 4)
    es = 2 if case["dtype"] == "bf16" else 4
    drawn = case["steps"] if case["call"] == "generate" else 0
    state = sum(min(n, (cfg.filter_width - 1) * d) for d in cfg.dilations) * B * cfg.channels * es
    return {"bytes": params + B * ((n - drawn) * (4 + 4 * cfg.n_classes) + drawn * 8)
            + (0 if case["call"] == "teacher" else state),
            "flops": B * n * cfg.flops_per_sample()}


def tolerance(case):
    if case["dtype"] == "bf16":
        # operand-rounding flips compound per layer: correct kernels of the same reading lie ~5e-3 apart
        return {"rel": 0.02, "max": 0.2}
    # float32 sums in another order: ~1e-6 apart; a draw next to a CDF boundary may fall on either side
    return {"rel": 5e-6, "max": 5e-5, "differ": 0.01}


def _forward(w, cfg, tokens):
    """Logits [B][T][Q] in 64 bits after consuming tokens [B][T] from zero queues: the dilated causal
    convolutions over the whole sequence."""
    def t(a):
        return torch.from_numpy(a).cuda().double()

    B, T = tokens.shape
    C = cfg.channels
    x = t(w.embed).t()[tokens.long()] + t(w.embed_b)
    skip = None
    for l, d in enumerate(cfg.dilations):
        conv, last = t(w.conv[l]), cfg.filter_width - 1
        a = x @ conv[:, :, last].t() + t(w.conv_b[l])
        for k in range(last):
            lag = (last - k) * d
            if lag < T:
                a[:, lag:] += x[:, :T - lag] @ conv[:, :, k].t()
        if cfg.kind == W.GATED:
            z = torch.tanh(a[..., :C]) * torch.sigmoid(a[..., C:])
            s = z @ t(w.skip[l]).t() + t(w.skip_b[l])
            skip = s if skip is None else skip.add_(s)
            x = x + z @ t(w.res[l]).t() + t(w.res_b[l])
        else:
            x = torch.relu(a) if cfg.kind == W.RELU else x + torch.relu(a)
    if cfg.kind == W.GATED:
        x = torch.relu(torch.relu(skip) @ t(w.head).t() + t(w.head_b))
    return x @ t(w.out).t() + t(w.out_b)


def exact(case, seed):
    """The 64-bit evaluation of the model as its weights define it (no intermediate rounding)."""
    cfg, w = _config(case), _weights(case, seed)
    seq, _ = _inputs(case, seed)
    if case["call"] != "teacher":  # the pending input comes first: after a reset the seed class
        first = torch.full((seq.shape[0], 1), cfg.seed_input, dtype=seq.dtype, device=seq.device)
        seq = torch.cat([first, seq[:, :-1]], 1)
    # stream by stream slices keep the 64-bit rows within a few GB
    per = max(1, (1 << 18) // seq.shape[1])
    lg = torch.cat([_forward(w, cfg, seq[i:i + per]) for i in range(0, seq.shape[0], per)])
    if case["call"] == "generate":
        return {"logits": lg, "samples": None}
    if case["call"] == "steps":
        return [lg[:, i:i + 1] for i in range(case["steps"])]
    if case["call"] == "prime":
        return {"prefix": lg[:, :case["prefix"]], "steps": lg[:, case["prefix"]:]}
    return lg
