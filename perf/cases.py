"""Decode calls of the engine over the range it is used in: the work behind each case, from one
short utterance of a tiny model to 128 utterances of a Parakeet-shaped decoder.

A case is a dict of plain values:
  model    which decoder (MODELS below)
  decoder  "frame" (Algorithm 1), "label" (label looping) or "tdt"
  dtype    "fp32", or the bfloat16 mode with its streamed weights kept as "bf16", "e4m3" or "e2m1"
  B, T     utterances and padded frames; lengths are uniform on lo..T, longest first
  S        most labels per frame (max_symbols)
  logp     also ask for the winning logits and the log-probabilities of the labels

Everything a call needs but its inputs (weights, engine, output buffers) is made in prepare(),
as a serving program would keep it; run() is one decode call.
"""
from __future__ import annotations

import functools
import math
from dataclasses import dataclass
from typing import Dict, Tuple

import numpy as np
import torch

import paper_2406_03791_amd as pkg
from paper_2406_03791_amd import binding


@dataclass(frozen=True)
class Dims:
    F: int
    E: int
    H: int
    L: int
    J: int
    V1: int
    durations: Tuple[int, ...] = ()
    big_blanks: Tuple[int, ...] = ()

    @property
    def D(self) -> int:
        return len(self.durations)

    @property
    def blank(self) -> int:
        return self.V1 - 1

    @property
    def n_out(self) -> int:
        return self.V1 + len(self.durations) + len(self.big_blanks)


# The decoder shapes of the repository's configurations.  The biases give these weights the blank
# rate of a trained model (about 80-85 % of the joint evaluations; the tiny model is left as drawn);
# rate: labels per frame that come out.
_PARAKEET = dict(F=1024, E=640, H=640, J=640, V1=1025)
MODELS = {
    "tiny": (Dims(F=64, E=64, H=64, L=1, J=64, V1=17), dict(bias=0.0, tied=False, rate=2.0)),
    "small": (Dims(F=256, E=320, H=320, L=1, J=320, V1=257), dict(bias=2.35, tied=True, rate=0.25)),
    "parakeet": (Dims(L=2, **_PARAKEET), dict(bias=10.22, tied=True, rate=0.17)),
    "one_layer": (Dims(L=1, **_PARAKEET), dict(bias=8.47, tied=True, rate=0.17)),
    "tdt": (Dims(L=2, durations=(0, 1, 2, 3, 4), **_PARAKEET), dict(bias=7.97, tied=True, rate=0.08)),
    "multi_blank": (Dims(L=2, big_blanks=(2, 4), **_PARAKEET),
                    dict(bias=6.5, big_bias=(6.5, 6.3), tied=True, rate=0.13)),
}
FLAGS = {"fp32": 0, "bf16": pkg.RNNT_FLAG_BF16_ARITHMETIC,
         "e4m3": pkg.RNNT_FLAG_BF16_ARITHMETIC | pkg.RNNT_FLAG_FP8_WEIGHTS,
         "e2m1": pkg.RNNT_FLAG_BF16_ARITHMETIC | pkg.RNNT_FLAG_FP4_WEIGHTS}
CAP_PER_FRAME = 10      # room for labels per frame in the output buffers


def listed():
    def c(name, model, decoder, dtype, B, T, lo, S=10, logp=False):
        return dict(name=name, model=model, decoder=decoder, dtype=dtype, B=B, T=T, lo=lo, S=S, logp=logp)
    return [
        # the smallest call: launches and hand-overs only
        c("tiny_frame_b1", "tiny", "frame", "fp32", 1, 20, 20, S=3),
        # a small recogniser, a handful of utterances
        c("small_frame_b8", "small", "frame", "fp32", 8, 200, 100, S=5),
        # one utterance at a time: an interactive recogniser
        c("label_b1", "parakeet", "label", "fp32", 1, 500, 200),
        # a few short odd-sized segments (voice commands), with confidences
        c("label_b5_logp", "parakeet", "label", "fp32", 5, 137, 40, logp=True),
        # offline transcription in batches of 32, the benchmark's configuration, all three decoders
        c("frame_b32", "parakeet", "frame", "fp32", 32, 500, 200),
        c("label_b32", "parakeet", "label", "fp32", 32, 500, 200),
        c("tdt_b32", "tdt", "tdt", "fp32", 32, 500, 200),
        # a ragged batch of a model with big blanks
        c("multi_blank_b19", "multi_blank", "label", "fp32", 19, 333, 51),
        # the same models in the precision they are served in
        c("label_b32_bf16", "parakeet", "label", "bf16", 32, 500, 200),
        c("tdt_b57_e4m3", "tdt", "tdt", "e4m3", 57, 411, 97),
        # throughput: large batches
        c("label_b128", "parakeet", "label", "fp32", 128, 500, 200),
        c("frame_b128", "parakeet", "frame", "fp32", 128, 500, 200),
    ]


def draw(rng):
    model = rng.choice(["tiny", "small", "parakeet", "parakeet", "parakeet", "one_layer", "tdt", "tdt",
                        "multi_blank"])
    decoder = {"tdt": "tdt", "multi_blank": "label"}.get(model) or rng.choice(["frame", "label"])
    dtype = "fp32"
    if model not in ("tiny", "small"):
        dtype = rng.choice(["fp32", "fp32", "fp32", "bf16", "bf16", "e4m3", "e2m1"])
    # (in the bfloat16 mode a rounded operand can differ by a whole step between two correct
    # summation orders, and then a row decodes differently from there on: a share of the rows of
    # a batch does, which says something of a batch and nothing of one or two utterances)
    lo_b = 1 if dtype == "fp32" else 8
    B = int(round(math.exp(rng.uniform(math.log(lo_b), math.log(128)))))
    T = int(round(math.exp(rng.uniform(math.log(20), math.log(500)))))
    lo = max(1, int(T * rng.uniform(0.1, 0.9)))
    S = {"tiny": 3, "small": 5}.get(model, 10)
    logp = dtype == "fp32" and B <= 8 and rng.random() < 0.5
    return dict(model=model, decoder=decoder, dtype=dtype, B=B, T=T, lo=lo, S=S, logp=logp)


class Model:
    """What the engine takes: dims and a name -> array table."""

    def __init__(self, dims: Dims, arrays: Dict[str, np.ndarray]):
        self.dims, self._arrays = dims, arrays

    def arrays(self):
        return self._arrays


@functools.lru_cache(maxsize=4)
def the_model(name: str, dtype: str) -> Model:
    """Weights uniform on +-0.1; the tied models carry the structure of a trained transducer
    (an emitted label lowers its own logit): the embedding of a label opposes its output row, and
    cell candidate and prediction-side projection pass that direction on."""
    d, kw = MODELS[name]
    g = np.random.default_rng(sorted(MODELS).index(name) + 17)
    U = lambda *shape: (g.random(shape, dtype=np.float32) - np.float32(0.5)) * np.float32(0.2)  # noqa: E731
    a = {"emb": U(d.V1, d.E)}
    a["emb"][d.blank] = 0.0
    for l in range(d.L):
        a[f"w_ih{l}"], a[f"w_hh{l}"] = U(4 * d.H, d.E if l == 0 else d.H), U(4 * d.H, d.H)
        a[f"b_ih{l}"], a[f"b_hh{l}"] = U(4 * d.H), U(4 * d.H)
    a["w_enc"], a["b_enc"], a["w_pred"], a["b_pred"] = U(d.J, d.F), U(d.J), U(d.J, d.H), U(d.J)
    a["w_out"], a["b_out"] = U(d.n_out, d.J), U(d.n_out)
    a["b_out"][d.blank] += np.float32(kw["bias"])
    for i, b in enumerate(kw.get("big_bias", ())):
        a["b_out"][d.V1 + i] += np.float32(b)
    if kw["tied"]:
        eye = np.eye(d.H, dtype=np.float32)
        a["emb"][:d.blank] -= np.float32(5.0) * a["w_out"][:d.blank]
        for l in range(d.L):
            a[f"w_ih{l}"][2 * d.H:3 * d.H] += np.float32(2.0) * eye
        a["w_pred"] += np.float32(5.0) * eye
    quantise = {"e4m3": pkg.rnnt_quantize_rows_e4m3, "e2m1": pkg.rnnt_quantize_blocks_e2m1}.get(dtype)
    if quantise:
        for key in ["w_pred", "w_out"] + [f"w_hh{l}" for l in range(d.L)] + [f"w_ih{l}" for l in range(1, d.L)]:
            a[key] = quantise(a[key])[0]
    return Model(d, a)


def prepare(case, seed):
    """Engine and buffers for the case, and a batch of encoder outputs ~ N(0, 1) of ragged lengths."""
    B, T, d = case["B"], case["T"], MODELS[case["model"]][0]
    engine = pkg.Engine(the_model(case["model"], case["dtype"]), B, T, device="cuda:0", flags=FLAGS[case["dtype"]])
    g = torch.Generator(device="cuda").manual_seed(seed)
    enc = torch.randn((B, T, d.F), generator=g, device="cuda", dtype=torch.float32)
    lens = torch.randint(case["lo"], T + 1, (B,), generator=g, device="cuda", dtype=torch.int32)
    lens = lens.sort(descending=True).values.contiguous()
    # labels, frames (and durations) and counts in one buffer, so that one copy brings a result
    # to the host; -1 beyond an utterance's last label
    cap = CAP_PER_FRAME * T
    n_tab = 3 if d.D else 2
    ints = torch.zeros(n_tab * B * cap + B, device="cuda", dtype=torch.int32)
    floats = torch.zeros((2, B, cap), device="cuda", dtype=torch.float32) if case["logp"] else None
    return dict(case=case, engine=engine, enc=enc, lens=lens, cap=cap, ints=ints, floats=floats,
                tables=[ints[i * B * cap:(i + 1) * B * cap] for i in range(n_tab)], counts=ints[n_tab * B * cap:])


def run(state):
    c, eng = state["case"], state["engine"].handle
    tab, fl = state["tables"], state["floats"]
    if fl is not None:
        binding.rnnt_engine_set_logp_output(eng, fl[1])
    stream = torch.cuda.current_stream().cuda_stream
    args = (eng, state["enc"], state["lens"], c["B"], c["T"], c["S"], tab[0], state["counts"], state["cap"], tab[1],
            fl[0] if fl is not None else None)
    if c["decoder"] == "tdt":
        binding.tdt_label_looping_decode(*args, tab[2], stream=stream)
    elif c["decoder"] == "label":
        binding.rnnt_label_looping_decode(*args, stream=stream)
    else:
        binding.rnnt_greedy_decode(*args, stream=stream)
    return state["ints"] if fl is None else {"ints": state["ints"], "logits": fl[0], "logps": fl[1]}


def work(case):
    """Frames read, weights read and outputs written once; the products of the projection, of one
    prediction step per label and of one joint evaluation per frame and per label."""
    d, kw = MODELS[case["model"]]
    frames = case["B"] * (case["lo"] + case["T"]) / 2
    labels = kw["rate"] * frames + case["B"]
    size = {"fp32": 4, "bf16": 2, "e4m3": 1, "e2m1": 0.5}[case["dtype"]]
    lstm = d.L * 4 * d.H * d.H + (d.L - 1) * 4 * d.H * d.H
    streamed = lstm + d.J * d.H + d.n_out * d.J
    out = case["B"] * case["T"] * CAP_PER_FRAME * 4 * ((3 if d.D else 2) + (2 if case["logp"] else 0))
    return {"bytes": frames * d.F * 4 + streamed * size + d.J * d.F * 4 + labels * 4 * d.H * 4 + out,
            "flops": 2.0 * (frames * d.F * d.J + labels * (lstm + d.J * d.H) + (frames + labels) * d.n_out * d.J)}


def tolerance(case):
    """Labels are integers: another summation order gives the same ones except where two logits
    tie to within rounding, and an utterance with such a tie may go on differently.  About 1.3 % of
    the entries of an utterance's tables are labels (a tied model).  fp32: one utterance of the call (ties are
    rare); bfloat16 mode: under half of them (operands are rounded, so sums that differ in the
    last bits can differ by a bfloat16 step afterwards).  Scores are 32-bit sums of 640 products."""
    differ = min(0.01, 0.013 / case["B"]) if case["dtype"] == "fp32" else 0.006
    return {"rel": 5e-5 if case["logp"] else 0.0, "differ": differ}
