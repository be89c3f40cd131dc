"""The training steps whose time this repository is judged by: what a case is, how its inputs are made, one pass.

A pass is one call of `mslt_train_step` (Section 3.2 of the paper: forward through the frozen and the trainable
layers, masked-LM loss, backward through the trainable part, optimizer update).  That is the one hot call of a
training run: `schedule.py` drives a whole run through it and nothing else in a run repeats.  The batch lies on
the GPU, as `Model.device_batch` leaves it; with dropout a pass first advances the dropout step, as a run does.

The cases cover the ranges a user meets: the three model shapes of `synth.py`; every stage of the schedule (first
stage and joint retraining with embeddings, middle and final stages with a frozen prefix); one sequence up to
16384 tokens; sequence lengths up to 512, the multiples of 128 of the paper's own runs and the lengths in between
that dynamic padding gives; full and ragged batches; bf16 and fp32 mode; Adam and LAMB; dropout, the next-sentence
head and the grouped variant on and off.
"""
import math

import torch

from paper_2011_13635_amd import binding, synth

_SHAPES = {"tiny": synth.tiny_shape, "base": synth.bert_base_shape, "large": synth.bert_large_shape}


def _case(name, model, frozen, trainable, batch, seq, *, ragged=False, fp32=False, lamb=True, dropout=0.0, nsp=False, group=1):
    """frozen + trainable layers of `model`; the embedding block trains when nothing is frozen."""
    return {"name": name, "model": model, "frozen": frozen, "trainable": trainable, "batch": batch, "seq": seq,
            "ragged": ragged, "fp32": fp32, "lamb": lamb, "dropout": dropout, "nsp": nsp, "group": group}


def listed():
    return [
        # the smallest step: a model of test size, where launches and host work are what counts
        _case("tiny_stage_4x64", "tiny", 2, 1, 4, 64, lamb=False),
        # fp32 mode at an odd size with everything trainable: how a change of the training recipe is checked
        _case("tiny_fp32_all_11x50", "tiny", 0, 3, 11, 50, ragged=True, fp32=True),
        # one sequence on BERT-Base: the smallest batch of a real model
        _case("base_final_1x128", "base", 9, 3, 1, 128, lamb=False),
        # fp32 mode on BERT-Base: the reference run that bf16 training is compared with
        _case("base_stage2_fp32_8x128", "base", 3, 3, 8, 128, fp32=True, lamb=False),
        # first stage of the Base schedule as trained: embeddings and dropout on
        _case("base_first_32x128", "base", 0, 3, 32, 128, dropout=0.1),
        # second stage of the Base schedule, the plain step
        _case("base_stage2_64x128", "base", 3, 3, 64, 128, lamb=False),
        # final stage with both objectives and dropout, as BERT is trained
        _case("base_final_nsp_64x128", "base", 9, 3, 64, 128, dropout=0.1, nsp=True),
        # a batch padded to its longest sequence: neither the length nor the rows are round numbers
        _case("base_final_ragged_27x203", "base", 9, 3, 27, 203, ragged=True, dropout=0.1),
        # final stage on the long sequences of the last tenth of the run
        _case("base_final_16x512", "base", 9, 3, 16, 512, lamb=False),
        # grouped variant (Section 3.3): three layers share one parameter set
        _case("base_grouped_64x128", "base", 9, 3, 64, 128, group=3),
        # the headline of bench.py: final stage of the BERT-Large schedule
        _case("large_final_64x128", "large", 18, 6, 64, 128),
        # joint retraining of BERT-Large on long sequences: the largest step
        _case("large_retrain_32x512", "large", 0, 24, 32, 512),
    ]


def draw(rng):
    """One more case of the same ranges; never more work than large_retrain_32x512."""
    model = rng.choices(["tiny", "base", "large"], [2, 6, 3])[0]
    fp32 = model != "large" and rng.random() < (0.4 if model == "tiny" else 0.12)
    group = 3 if model == "base" and rng.random() < 0.12 else 1
    per_stage = {"tiny": 1, "base": 3, "large": 6}[model]
    stage = rng.randint(1, 4)                         # one of four stages, or the joint retraining of so many layers
    all_trainable = stage == 1 or rng.random() < 0.15
    frozen = 0 if all_trainable else (stage - 1) * per_stage
    trainable = stage * per_stage if all_trainable else per_stage
    if rng.random() < 0.5:
        seq = 128 * rng.choice([1, 1, 1, 2, 3, 4])
    else:
        seq = round(math.exp(rng.uniform(math.log(24), math.log(512))))
    most = {"tiny": 8192, "base": 16384, "large": 16384}[model] if not fp32 else {"tiny": 4096, "base": 1536}[model]
    tokens = math.exp(rng.uniform(math.log(128), math.log(most)))
    batch = max(1, min(round(tokens / seq), most // seq))
    case = _case("", model, frozen, trainable, batch, seq, ragged=rng.random() < 0.4, fp32=fp32, lamb=rng.random() < 0.6,
                 dropout=0.1 if rng.random() < 0.5 else 0.0, nsp=rng.random() < 0.25, group=group)
    del case["name"]
    return case


def _shape(case):
    base = _SHAPES[case["model"]](case["frozen"] + case["trainable"]).as_dict()
    base.update(nsp=case["nsp"], layers_per_group=case["group"])
    return synth.ModelShape(**base)


def _weights(table, seed):
    """Packed start weights, as synth.make_weights distributes them (matrices and tables N(0, 0.02), gains 1, the
    rest 0), but drawn on the GPU: a BERT-Large stack has 335 million of them."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    parts = []
    for name, _, rows, cols, _, _, count in table:
        if cols > 1:
            parts.append(torch.randn(count, generator=gen, device="cuda", dtype=torch.float32) * 0.02)
        else:
            parts.append(torch.full((count,), 1.0 if name.endswith("_g") else 0.0, device="cuda"))
    return torch.cat(parts).cpu().numpy()


def prepare(case, seed):
    shape = _shape(case)
    cfg = binding.make_config(shape, case["batch"], case["seq"], 0 if case["fp32"] else 1,
                              max_trainable_layers=case["trainable"])
    model = binding.Model(cfg)
    model.mslt_load_params(_weights(model.table, seed))
    batch = model.device_batch(synth.make_batch(shape, case["batch"], case["seq"], seed=seed + 1, ragged=case["ragged"]))
    opt = binding.lamb() if case["lamb"] else binding.adam(lr=1e-4)
    # what a step writes, as views of the model's own arenas: gradients layer by layer (their scales differ), weights
    # and both moments of each trained block
    param, grad = (a.view(torch.float32) for a in model.arenas[:2])
    m1, m2 = model.arenas[2].view(torch.float32).chunk(2)
    spans, sets = {}, case["frozen"] // case["group"]
    for _, layer, _, _, _, offset, count in model.table:
        if layer == -1 and case["frozen"] > 0 or 0 <= layer < sets:
            continue
        block = {-1: "emb", -2: "head"}.get(layer, "layer%d" % layer)
        lo, hi = spans.get(block, (offset, offset))
        spans[block] = (lo, offset + count)
    layers = [v for k, v in spans.items() if k.startswith("layer")]
    blocks = {"layers": (layers[0][0], layers[-1][1]), **{k: v for k, v in spans.items() if not k.startswith("layer")}}
    out = {"grad." + k: grad[lo:hi] for k, (lo, hi) in spans.items()}
    for k, (lo, hi) in blocks.items():
        out.update({"weights." + k: param[lo:hi], "m." + k: m1[lo:hi], "v." + k: m2[lo:hi]})
    return {"model": model, "batch": batch, "opt": opt, "frozen": case["frozen"], "trainable": case["trainable"],
            "dropout": case["dropout"], "step": 0, "seed": seed, "out": out}


def run(state):
    model = state["model"]
    if state["dropout"]:
        model.mslt_set_dropout(state["dropout"], state["seed"], state["step"])
        state["step"] += 1
    loss = model.mslt_train_step(state["frozen"], state["trainable"], state["frozen"] == 0, state["batch"], state["opt"])
    return {"loss": loss, **state["out"]}


def work(case):
    s = _shape(case)
    H, F, V, S, B = s.hidden, s.ffn, s.vocab, case["seq"], case["batch"]
    T, f, k = B * S, case["frozen"], case["trainable"]
    emb = f == 0
    M = B * synth.n_masked_for_length(round(0.75 * S) if case["ragged"] else S)     # predicted positions
    Mt = M + (B if case["nsp"] else 0)             # rows of the top layer's output that get a gradient
    qkv, wo, ffn, attn = 6.0 * H * H, 2.0 * H * H, 4.0 * H * F, 4.0 * S * H           # forward FLOPs per token
    flops = (f + k) * T * (qkv + wo + ffn + attn)
    flops += (k - 1) * T * 2 * (wo + ffn) + Mt * 2 * (wo + ffn)                       # weight and data gradients,
    flops += k * T * (2 * qkv + 2 * attn) - (0 if emb else T * qkv)                   # none below the trained part
    flops += M * (3 * 2.0 * H * H + (3 if emb else 2) * 2.0 * H * V)                  # head and tied decoder
    if case["nsp"]:
        flops += 3 * 2.0 * B * H * (H + 2)
    # bytes: frozen weights once as the products read them; of trained tensors weights and moments in and out and the
    # gradient out; the batch; the rows of the embedding tables that are looked up
    layer = 4 * H * H + 2 * H * F + 9 * H + F
    tables = (V + s.max_pos + s.type_vocab) * H + 2 * H
    head = H * H + 3 * H + V + (H * H + 3 * H + 2 if case["nsp"] else 0)
    trained = k // case["group"] * layer + head + (tables if emb else 0)
    fixed = f // case["group"] * layer + (0 if emb else V * H)
    esz = 4 if case["fp32"] else 2
    return {"bytes": trained * 28.0 + fixed * esz + T * (16.0 + 8.0 * H), "flops": flops}


def tolerance(case):
    """Four times what was seen over two steps: fp32 mode against the float64 oracle (largest relative error of any
    output 3.7e-6, largest single difference 5e-5 of the tensor's scale, tiny and Base), bf16 mode against fp32 mode
    (1.4e-2 and 0.6, the latter in the embedding gradient, most rows of which are zero)."""
    return {"rel": 2e-5, "max": 5e-4} if case["fp32"] else {"rel": 0.03, "max": 0.95}
