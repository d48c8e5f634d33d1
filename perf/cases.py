"""Performance cases of the L2L relay-execution library, through its public entry points (binding.py, trainer.py).

Three kinds of work, which is what a program does with this library:

 - "layer": the passes of one resident encoder layer over the U micro-batches of a mini-batch (l2l_layer_fwd_stats,
   l2l_layer_bwd_stats, l2l_grad_drain): the calls a step driver makes once per layer and direction.  The layer's weights
   have been staged; the upstream gradient, which the backward call turns into dL/dX in place, is copied in from where
   the layer above left it.
 - "embed_head": the first and the last resident "layer": embedding, tied LM head with cross-entropy, embedding
   backward, and the drain of their gradients.
 - "step": one whole training step of a small model through the step driver: stages, forward, head, backward, drains, and
   Adam on the host.

The widths are those of the five named workloads (l2l_synth.WORKLOADS) and generic ones around them; a run returns every
output whole: boundary activations, kept statistics, dL/dX, every parameter gradient, and a step's loss and gradients (its
updated weights are what the next pass computes with).
"""
import ctypes
import math

import torch

from paper_2002_05645_amd import binding as B
from paper_2002_05645_amd.trainer import L2LTrainer

TORCH = {"bf16": torch.bfloat16, "fp16": torch.float16, "fp32": torch.float32}
LN_EPS = 1e-12
VOCAB = 30522      # of the named workloads
LABELLED = 0.15    # share of positions that carry a label, likewise


def layer(name, direction, hidden, heads, ffn, seq, ubatch, num_ubatches, dtype, drain="fp32"):
    return dict(name=name, path="layer", direction=direction, hidden=hidden, heads=heads, ffn=ffn, seq=seq, ubatch=ubatch,
                num_ubatches=num_ubatches, dtype=dtype, drain=drain)


def listed():
    return [
        # The smallest whole call: a training step of the tiny workload in fp32, the configuration of the library's smoke
        # run: launches, event waits and host work count, arithmetic does not.
        dict(name="step_tiny_fp32", path="step", layers=2, hidden=128, heads=2, ffn=512, seq=64, vocab=1000, ubatch=4,
             num_ubatches=4, dtype="fp32", labelled=1.0, eager=False),
        # An ordinary whole step: the BERT-Base workload at a depth of three layers, optimizer running eagerly per layer.
        dict(name="step_base_bf16", path="step", layers=3, hidden=768, heads=12, ffn=3072, seq=128, vocab=VOCAB, ubatch=16,
             num_ubatches=8, dtype="bf16", labelled=LABELLED, eager=True),
        # The smallest layer call: the forward pass of a single short sequence (evaluation at batch size one).
        layer("fwd_one_sequence_bf16", "fwd", 1024, 16, 4096, 64, 1, 1, "bf16"),
        # One micro-batch per layer visit, the left end of the paper's micro-batch sweep (Tables 3 and 4), with the bf16
        # drains that one uses there (fp32 ones take longer than the layer).
        layer("layer_large_u1_bf16", "both", 1024, 16, 4096, 128, 32, 1, "bf16", drain="bf16"),
        # The headline workload's two calls: BERT-Large, eight micro-batches of 32 sequences of 128 tokens.
        layer("fwd_large_bf16", "fwd", 1024, 16, 4096, 128, 32, 8, "bf16"),
        layer("bwd_large_bf16", "bwd", 1024, 16, 4096, 128, 32, 8, "bf16"),
        # The long-sequence workload: BERT-Large at 512 tokens, sixteen micro-batches of four sequences.
        layer("layer_large_s512_bf16", "both", 1024, 16, 4096, 512, 4, 16, "bf16"),
        # The paper's own device precision (loss-scaled FP16) on the BERT-Base workload.
        layer("layer_base_fp16", "both", 768, 12, 3072, 128, 16, 8, "fp16"),
        # Ragged: head width 96, a sequence length that is no multiple of 16, odd micro-batches, nothing a multiple of a tile.
        layer("layer_ragged_bf16", "both", 1152, 12, 4616, 200, 5, 7, "bf16"),
        # Full precision, the mode that training is checked against: BERT-Base width, fp32 throughout.
        layer("layer_base_fp32", "both", 768, 12, 3072, 128, 16, 2, "fp32"),
        # Embedding and LM head of the headline workload, forward and backward, their 32 million gradients drained in bf16.
        dict(name="embed_head_large_bf16", path="embed_head", hidden=1024, heads=16, ffn=4096, seq=128, ubatch=32, num_ubatches=8,
             vocab=VOCAB, dtype="bf16", labelled=LABELLED, drain="bf16"),
        # The largest: a layer of the deep-wide workload (453 million parameters), gradients sent to the host rounded to
        # bf16 as the option for link-bound models has it.
        layer("layer_deep_wide_bf16", "both", 6144, 48, 24576, 128, 8, 8, "bf16", drain="bf16"),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    """One more case of the same ranges: widths 128 to 2048 with head widths 32 to 128 (64 most often), sequences of 8
    to 512 tokens (any multiple of 8), 64 to 32768 tokens per mini-batch in 1 to 16 micro-batches, the three formats."""
    kind = rng.choice(["layer"] * 8 + ["embed_head", "step"])
    dtype = rng.choice(["bf16"] * 6 + ["fp16"] * 2 + ["fp32"] * 2)
    while True:
        d = rng.choice([64] * 5 + [32, 80, 96, 128])
        hidden = 8 * round(_log_uniform(rng, 128, 2048) / 8)
        heads = max(1, round(hidden / d))
        hidden = heads * d
        if hidden > 2048:
            continue
        ffn = rng.choice([4 * hidden, 4 * hidden, 8 * round(rng.uniform(2.5, 4.5) * hidden / 8)])
        seq = rng.choice([32, 64, 128, 128, 256, 512, 8 * round(_log_uniform(rng, 8, 512) / 8)])
        tokens = _log_uniform(rng, 64, 32768)
        num_ubatches = rng.choice([1, 2, 4, 8, 16, rng.randint(1, 16)])
        ubatch = round(tokens / (seq * num_ubatches))
        if not 1 <= ubatch <= 64 or ubatch * seq * num_ubatches > 40000:
            continue
        # fp32 runs at a sixteenth of the 16-bit formats' arithmetic rate: smaller mini-batches, as a check run has
        if dtype == "fp32" and ubatch * seq * num_ubatches > 4096:
            continue
        break
    shape = dict(hidden=hidden, heads=heads, ffn=ffn, seq=seq, ubatch=ubatch, num_ubatches=num_ubatches, dtype=dtype)
    if kind == "layer":
        direction = rng.choice(["fwd", "bwd", "both", "both"])
        return dict(path="layer", direction=direction, drain="bf16" if direction != "fwd" and dtype == "bf16" and rng.random() < 0.25 else "fp32", **shape)
    vocab = 2 * round(_log_uniform(rng, 1000, VOCAB) / 2)
    if kind == "embed_head":
        return dict(path="embed_head", vocab=vocab, labelled=1.0 if vocab < 8000 and rng.random() < 0.5 else LABELLED,
                    drain="bf16" if dtype == "bf16" and rng.random() < 0.5 else "fp32", **shape)
    # whole steps stay small: their parameters live on the host, optimizer state and all
    layers = rng.randint(1, 4)
    while layers > 1 and layers * hidden * hidden * 12 > 40e6:
        layers -= 1
    return dict(path="step", layers=layers, vocab=min(vocab, 8000), labelled=rng.choice([LABELLED, 1.0]), eager=rng.random() < 0.5, **shape)


# One compute stream and one copy stream for the process, as a training program has them; torch's current stream is the
# compute stream, so that the program's own torch operations are ordered with the library's kernels.
_streams = []


def _compute_and_copy():
    if not _streams:
        _streams.extend([torch.cuda.Stream(), torch.cuda.Stream()])
    torch.cuda.set_stream(_streams[0])
    return _streams[0].cuda_stream, _streams[1].cuda_stream


class State:
    """What a program holds between calls; gives the library's context or the step driver back when it is dropped."""

    def __init__(self, case):
        self.case = case
        self.owned = None

    def __del__(self):
        if self.owned is not None:
            self.owned.close()
            self.owned = None


class Outputs(dict):
    """A run's outputs; a step's gradients are views of the driver's host buffers, which live as long as these."""
    state = None


def _shapes(case):
    H, F = case["hidden"], case["ffn"]
    return {"Wqkv": (H, 3 * H), "bqkv": (3 * H,), "Wo": (H, H), "bo": (H,), "g1": (H,), "be1": (H,), "W1": (H, F), "b1": (F,),
            "W2": (F, H), "b2": (H,), "g2": (H,), "be2": (H,)}


def _embed_shapes(case):
    H, V, S = case["hidden"], case["vocab"], case["seq"]
    return {"E": (V, H), "P": (S, H), "ge": (H,), "be": (H,), "bv": (V,)}


def _fill_block(block, layout, gen):
    """N(0, 0.02) in every tensor, gains around one, padding zero"""
    for name, (off, n) in layout.items():
        block[off:off + n].normal_(0.0, 0.02, generator=gen)
        if name in ("g1", "g2", "ge"):
            block[off:off + n] += 1.0


def _pinned_views(layout, total, dtype):
    """landing buffer for drained gradients, and its tensors by name"""
    land = torch.zeros(total, dtype=dtype).pin_memory()
    return land, {name: land[off:off + n] for name, (off, n) in layout.items()}


def _tokens_and_labels(case, gen):
    shape = (case["num_ubatches"], case["ubatch"], case["seq"])
    tok = torch.randint(0, case["vocab"], shape, dtype=torch.int32, device="cuda", generator=gen)
    lab = torch.randint(0, case["vocab"], shape, dtype=torch.int32, device="cuda", generator=gen)
    keep = torch.rand(shape, device="cuda", generator=gen) < case["labelled"]
    keep.view(-1)[0] = True
    return tok, torch.where(keep, lab, torch.full_like(lab, -1))


def prepare(case, seed):
    return {"layer": _prepare_layer, "embed_head": _prepare_embed_head, "step": _prepare_step}[case["path"]](case, seed)


def _prepare_layer(case, seed):
    compute, copy = _compute_and_copy()
    gen = torch.Generator(device="cuda").manual_seed(seed)
    dt = TORCH[case["dtype"]]
    cfg = B.make_config(case["hidden"], case["heads"], case["ffn"], case["seq"], case["ubatch"], case["num_ubatches"], case["dtype"], LN_EPS)
    st = State(case)
    st.ctx = st.owned = B.Context(cfg, compute, copy)
    layout, total = B.layer_layout(cfg), B.lib().l2l_layer_packed_elems(ctypes.byref(cfg))
    block = torch.zeros(total, dtype=dt, device="cuda")
    _fill_block(block, layout, gen)
    host = torch.empty(total, dtype=dt, pin_memory=True)
    host.copy_(block)
    del block
    st.ctx.param_stage(0, host, 0)
    st.ctx.sync()
    tokens = case["num_ubatches"] * case["ubatch"] * case["seq"]
    acts = (case["num_ubatches"], case["ubatch"], case["seq"], case["hidden"])
    # boundary activations are LayerNorm outputs; upstream gradients of size 1e-3, times the loss scale in fp16
    st.x = torch.randn(acts, device="cuda", generator=gen).to(dt)
    st.y = torch.empty_like(st.x)
    st.rstd = torch.empty(tokens, dtype=torch.float32, device="cuda")
    if case["direction"] != "fwd":
        st.dy_above = (torch.randn(acts, device="cuda", generator=gen) * (1.0 if case["dtype"] == "fp16" else 1e-3)).to(dt)
        st.dy = torch.empty_like(st.dy_above)
        if case["drain"] != "fp32":
            st.ctx.set_drain_dtype(case["drain"])
        st.land, st.grads = _pinned_views(layout, total, TORCH[case["drain"]])
    if case["direction"] == "bwd":
        st.ctx.layer_fwd_stats(0, 0, st.x, st.y, st.rstd)
    st.ctx.sync()
    return st


def _prepare_embed_head(case, seed):
    compute, copy = _compute_and_copy()
    gen = torch.Generator(device="cuda").manual_seed(seed)
    dt = TORCH[case["dtype"]]
    cfg = B.make_config(case["hidden"], case["heads"], case["ffn"], case["seq"], case["ubatch"], case["num_ubatches"], case["dtype"], LN_EPS,
                        vocab=case["vocab"])
    st = State(case)
    st.ctx = st.owned = B.Context(cfg, compute, copy)
    if case["dtype"] == "fp16":
        st.ctx.set_loss_scale(2.0 ** 15)
    layout, total = B.embed_layout(cfg), B.lib().l2l_embed_packed_elems(ctypes.byref(cfg))
    block = torch.zeros(total, dtype=dt, device="cuda")
    _fill_block(block, layout, gen)
    host = torch.empty(total, dtype=dt, pin_memory=True)
    host.copy_(block)
    st.ctx.embed_stage(host)
    st.ctx.sync()
    acts = (case["num_ubatches"], case["ubatch"], case["seq"], case["hidden"])
    st.tokens, st.labels = _tokens_and_labels(case, gen)
    st.x_last = torch.randn(acts, device="cuda", generator=gen).to(dt)      # the last layer's output
    st.dx0 = (torch.randn(acts, device="cuda", generator=gen) * (1.0 if case["dtype"] == "fp16" else 1e-3)).to(dt)   # dL/d(first layer's input)
    st.x0, st.dy = torch.empty_like(st.x_last), torch.empty_like(st.x_last)
    st.loss = torch.zeros(1, dtype=torch.float32, device="cuda")
    if case["drain"] != "fp32":
        st.ctx.set_drain_dtype(case["drain"])
    st.land, st.grads = _pinned_views(layout, total, TORCH[case["drain"]])
    st.ctx.sync()
    return st


def _prepare_step(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    st = State(case)
    st.trainer = st.owned = L2LTrainer(layers=case["layers"], hidden=case["hidden"], heads=case["heads"], ffn=case["ffn"], seq=case["seq"],
                                       vocab=case["vocab"], ubatch=case["ubatch"], num_ubatches=case["num_ubatches"], dtype=case["dtype"],
                                       eager=case["eager"])
    host = torch.Generator().manual_seed(seed)

    def tensors(shapes):
        return {k: (torch.randn(s, generator=host) * 0.02 + (1.0 if k in ("g1", "g2", "ge") else 0.0)).numpy() for k, s in shapes.items()}

    st.trainer.load_params(tensors(_embed_shapes(case)), [tensors(_shapes(case)) for _ in range(case["layers"])])
    st.tokens, st.labels = _tokens_and_labels(case, gen)
    st.grads = [st.trainer.eps.grad(b) for b in range(case["layers"] + 1)]
    torch.cuda.synchronize()
    return st


def run(st):
    case = st.case
    if case["path"] == "layer":
        c, direction = st.ctx, case["direction"]
        out = Outputs()
        if direction != "bwd":
            c.layer_fwd_stats(0, 0, st.x, st.y, st.rstd)
            out.update(y=st.y, rstd=st.rstd)
        if direction != "fwd":
            st.dy.copy_(st.dy_above)
            c.layer_bwd_stats(0, 0, st.x, st.y, st.rstd, st.dy)
            c.grad_drain(0, st.land)
            out.update(dx=st.dy, grads=st.grads)
        return out
    if case["path"] == "embed_head":
        c = st.ctx
        c.embed_fwd(st.tokens, st.x0)
        c.head_loss(st.x_last, st.labels, st.dy, st.loss)
        c.embed_bwd(st.tokens, st.dx0)
        c.embed_grad_drain(st.land)
        return Outputs(x0=st.x0, loss=st.loss, dy=st.dy, grads=st.grads)
    out = Outputs(loss=st.trainer.step(st.tokens, st.labels), grads=st.grads)
    out.state = st
    return out


def _layer_work(case):
    """(bytes, flops) of a layer's forward and of its backward pass with recompute (all but the FFN2 product)"""
    H, F, S, A = case["hidden"], case["ffn"], case["seq"], case["heads"]
    T = case["num_ubatches"] * case["ubatch"] * S
    es = 4 if case["dtype"] == "fp32" else 2
    params = 4 * H * H + 2 * H * F + 9 * H + F
    proj, attn = T * 2.0 * (4 * H * H + 2 * H * F), 4.0 * T * S * H
    fwd = (es * (params + 2.0 * T * H) + 4.0 * T, proj + attn)
    drain = 4 if case.get("drain", "fp32") == "fp32" else 2
    bwd = (es * (params + 4.0 * T * H) + 4.0 * T + drain * params, 2 * proj + 2.5 * attn + proj - T * 2.0 * H * F + attn)
    return fwd, bwd


def _embed_head_work(case):
    H, V, S = case["hidden"], case["vocab"], case["seq"]
    T = case["num_ubatches"] * case["ubatch"] * S
    es = 4 if case["dtype"] == "fp32" else 2
    rows = T * case["labelled"]
    params = V * H + S * H + 2 * H + V
    drain = 4 if case.get("drain", "fp32") == "fp32" else 2
    return es * (params + 4.0 * T * H) + 8.0 * T + drain * params, 6.0 * rows * V * H


def work(case):
    if case["path"] == "embed_head":
        b, f = _embed_head_work(case)
        return {"bytes": b, "flops": f}
    fwd, bwd = _layer_work(case)
    if case["path"] == "layer":
        parts = {"fwd": [fwd], "bwd": [bwd], "both": [fwd, bwd]}[case["direction"]]
        return {"bytes": sum(p[0] for p in parts), "flops": sum(p[1] for p in parts)}
    b, f = _embed_head_work(case)
    n = case["layers"]
    return {"bytes": b + n * (fwd[0] + bwd[0]), "flops": f + n * (fwd[1] + bwd[1])}


def tolerance(case):
    """About four times what is seen against the same pass in 64 bits on the same rounded inputs (layer: rel 5.7e-3, 6.2e-4
    and 1.4e-6, max 5.6e-2, 5.9e-3 and 1.1e-5 in bf16, fp16 and fp32; embedding and head: rel 2.8e-3, 3.0e-4 and 9.8e-7, max
    6.2e-3, 9.2e-4 and 6.5e-6), and for a step, whose second pass starts from weights that its first has updated, against
    steps that recompute the whole layer and that take attention as separate products (max 2.0e-1, 2.5e-2 and 3.3e-4, in the
    token rows of the embedding's gradient, most of which are small)."""
    rel = {"bf16": 2e-2, "fp16": 2.5e-3, "fp32": 1e-5}
    most = {"layer": {"bf16": 2e-1, "fp16": 2.5e-2, "fp32": 1e-4}, "embed_head": {"bf16": 2.5e-2, "fp16": 1e-2, "fp32": 3e-5},
            "step": {"bf16": 8e-1, "fp16": 1e-1, "fp32": 1.5e-3}}
    if case["path"] == "embed_head":
        rel = {"bf16": 1.1e-2, "fp16": 1.2e-3, "fp32": 1e-5}
    return {"rel": rel[case["dtype"]], "max": most[case["path"]][case["dtype"]]}
