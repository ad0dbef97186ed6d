"""The work a program has this library do, as cases that can be timed and compared.

A case is one call (or one fixed sequence of calls) of the binding on inputs that lie in device memory, with the
buffers and the workspace such a program keeps between calls.  Kinds:

  layer      one prefill layer step: attention, scores, selection, one gather (pyr_prefill_layer, or the merged call
             where hidden rows travel along, or the extended one with averaging weights and position ids)
  attention  the attention launch alone, with the row statistics the score pass needs
  score      the score pass alone, on row statistics that exist already
  select     the selection on given scores and the K/V gather that follows it, called one by one
  decode     the generation-phase update of a compressed cache

Lengths of a ragged batch come from the case itself ("lens": a seed), so every input seed has the same shapes.
Gathered rows are byte copies and are returned as 16-bit words.
"""
import math
import random

import torch

from paper_2405_12532_amd import binding


def listed():
    return [
        # a short prompt on a small model: launches and latency are all there is
        dict(name="layer-1x256-d64", kind="layer", n=1, lo=256, hi=256, hq=8, hkv=8, d=64, w=16, keep=50),
        # one prompt of a chat on a 7B-shaped layer, hidden rows and position ids travelling along
        dict(name="layer-1x2048", kind="layer", n=1, lo=2048, hi=2048, hq=32, hkv=32, d=128, w=64, keep=93, hidden=4096, pos=True),
        # one long document, grouped heads
        dict(name="layer-1x8192-gqa", kind="layer", n=1, lo=8192, hi=8192, hq=32, hkv=8, d=128, w=64, keep=80),
        # the batch throughput is quoted on: first layer of 64 prompts of 2k tokens
        dict(name="layer-64x2048", kind="layer", n=64, lo=2048, hi=2048, hq=32, hkv=32, d=128, w=64, keep=93, hidden=4096),
        # the same batch deep in the pyramid, where most of its layers have few tokens left
        dict(name="layer-64x359", kind="layer", n=64, lo=359, hi=359, hq=32, hkv=32, d=128, w=64, keep=93, hidden=4096),
        # prompts of any length in one batch on a 13B-shaped layer, recent rows weighted
        dict(name="layer-ragged32", kind="layer", n=32, lo=512, hi=8192, lens=4, hq=40, hkv=40, d=128, w=64, keep=60, weights=True,
             pos=True),
        # long inputs, many query heads on few key/value heads
        dict(name="layer-4x32768-gqa", kind="layer", n=4, lo=32768, hi=32768, hq=64, hkv=8, d=128, w=128, keep=50),
        # attention by itself on a handful of ragged prompts, d = 64
        dict(name="attention-ragged7-d64", kind="attention", n=7, lo=100, hi=3000, lens=7, hq=32, hkv=8, d=64, w=32, keep=50),
        # the score pass by itself (another attention kernel may have left the row statistics)
        dict(name="score-8x2048", kind="score", n=8, lo=2048, hi=2048, hq=32, hkv=32, d=128, w=64, keep=70),
        # selection and gather by themselves over long contexts
        dict(name="select-4x32768", kind="select", n=4, lo=32768, hi=32768, hq=64, hkv=8, d=128, w=128, keep=50),
        # generation: one conversation's cache, one token over its budget
        dict(name="decode-1x1537", kind="decode", n=1, lo=1537, hi=1537, hq=32, hkv=32, d=128, w=64, keep=99, pos=True),
        # generation: a serving batch
        dict(name="decode-64x2048", kind="decode", n=64, lo=2048, hi=2048, hq=32, hkv=32, d=128, w=64, keep=93),
    ]


_HEADS = [(8, 8, 64), (32, 8, 64), (12, 12, 64), (32, 32, 128), (40, 40, 128), (32, 8, 128), (64, 8, 128), (24, 24, 128)]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["layer", "layer", "layer", "attention", "score", "select", "decode", "decode"])
    hq, hkv, d = rng.choice(_HEADS)
    n = _log_int(rng, 1, 64)
    top = _log_int(rng, 100, 32768)
    top = max(64, min(top, 131072 // n))
    low = top if rng.random() < 0.5 else max(48, int(top * rng.uniform(0.1, 0.9)))
    case = dict(kind=kind, n=n, lo=low, hi=top, hq=hq, hkv=hkv, d=d, w=rng.choice([16, 32, 48, 64, 100, 128]), keep=rng.randint(40, 97))
    if low < top:
        case["lens"] = rng.randrange(1000)
    if kind in ("layer", "decode"):
        case["pos"] = rng.random() < 0.4
        case["weights"] = rng.random() < 0.3
    if kind == "layer" and rng.random() < 0.5:
        case["hidden"] = hq * d
    return case


def _lengths(case):
    if case["lo"] == case["hi"]:
        return [case["lo"]] * case["n"]
    rng = random.Random(case["lens"])
    return [rng.randint(case["lo"], case["hi"]) for _ in range(case["n"])]


def _keeps(case, lens):
    return [max(min(case["w"], S), (case["keep"] * S + 50) // 100) for S in lens]


class _Inputs:
    """The batch of a case in device memory: queries with a direction per head, keys that lie along it to a degree of
    their own (so that tokens differ in importance by orders of magnitude, as they do in a trained model)."""

    def __init__(self, case, seed):
        self.lens = _lengths(case)
        self.keeps = _keeps(case, self.lens)
        self.n, self.T, self.kept = case["n"], sum(self.lens), sum(self.keeps)
        self.hq, self.hkv, self.d, self.w = case["hq"], case["hkv"], case["d"], case["w"]
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(seed)
        off = [0]
        for S in self.lens:
            off.append(off[-1] + S)
        self.off = off
        self.off_h = torch.tensor(off, dtype=torch.int32)
        self.keep_h = torch.tensor(self.keeps, dtype=torch.int32)
        self.off_d, self.keep_d = self.off_h.cuda(), self.keep_h.cuda()
        self.shape = binding.make_shape(self.n, self.T, max(self.lens), self.hq, self.hkv, self.d)

    def normal(self, *size):
        return torch.randn(size, generator=self.gen, device="cuda")

    def directions(self):
        u = self.normal(self.hkv, self.d)
        return u / u.norm(dim=1, keepdim=True)

    def queries(self, rows, u):
        """[rows, hq, d] bf16"""
        q = self.normal(rows, self.hkv, self.hq // self.hkv, self.d)
        q += (0.35 * math.sqrt(self.d)) * u[None, :, None, :]
        return q.reshape(rows, self.hq, self.d).to(torch.bfloat16)

    def keys(self, u):
        k = self.normal(self.T, self.hkv, self.d)
        k += (3.0 * self.normal(self.T))[:, None, None] * u[None]
        return k.to(torch.bfloat16)

    def values(self):
        return self.normal(self.T, self.hkv, self.d).to(torch.bfloat16)

    def row_weights(self):
        return 0.25 + torch.rand(self.w, generator=self.gen, device="cuda")


def _scale(d):
    return 1.0 / math.sqrt(d)


def prepare(case, seed):
    x = _Inputs(case, seed)
    kind = case["kind"]
    s = dict(kind=kind, x=x)
    if kind == "select":
        # importances as the score pass leaves them: positive, spread over orders of magnitude, summing to one per sequence
        sc = torch.exp(1.2 * x.normal(x.T))
        for b in range(x.n):
            sc[x.off[b]:x.off[b + 1]] /= sc[x.off[b]:x.off[b + 1]].sum()
        s["scores"] = sc
        s["k"], s["v"] = x.values(), x.values()
    else:
        u = x.directions()
        s["k"] = x.keys(u)
        if kind == "decode":
            s["q"] = x.queries(x.n * x.w, u).reshape(x.n, x.w, x.hq, x.d)
        else:
            s["q"] = x.queries(x.T, u)
        if kind != "score":
            s["v"] = x.values()
    s["rw"] = x.row_weights() if case.get("weights") else None
    s["pos"] = s["pos_out"] = s["hidden"] = s["hidden_out"] = None
    if case.get("pos"):
        s["pos"] = torch.randint(0, 1 << 20, (x.T,), generator=x.gen, device="cuda", dtype=torch.int32)
        s["pos_out"] = torch.empty(x.kept, dtype=torch.int32, device="cuda")
    if case.get("hidden"):
        s["hidden"] = x.normal(x.T, case["hidden"]).to(torch.bfloat16)
        s["hidden_out"] = torch.empty(x.kept, case["hidden"], dtype=torch.bfloat16, device="cuda")
    if kind in ("layer", "attention"):
        s["out"] = torch.empty_like(s["q"])
    if kind == "attention":
        s["lse"] = torch.empty(x.T, x.hq, dtype=torch.float32, device="cuda")
        s["tile_map"] = torch.empty(x.n + 1, dtype=torch.int32, device="cuda")
    if kind == "score":
        s["lse"] = torch.zeros(x.T, x.hq, dtype=torch.float32, device="cuda")
        for b in range(x.n):
            r0, r1 = x.off[b], x.off[b + 1]
            L = min(x.w, r1 - r0)
            logits = _window_logits(s["q"][r1 - L:r1].float(), s["k"][r0:r1].float(), x)
            s["lse"][r1 - L:r1] = (torch.logsumexp(logits, dim=2) / math.log(2.0)).t()
    if kind in ("layer", "score", "decode"):
        s["scores"] = torch.empty(x.T, dtype=torch.float32, device="cuda")
    if kind in ("layer", "select", "decode"):
        s["kept"] = torch.empty(x.kept, dtype=torch.int32, device="cuda")
        s["out_off"] = torch.empty(x.n + 1, dtype=torch.int32, device="cuda")
        s["k_out"] = torch.empty(x.kept, x.hkv, x.d, dtype=torch.bfloat16, device="cuda")
        s["v_out"] = torch.empty_like(s["k_out"])
    if kind in ("layer", "decode"):
        size = binding.workspace_bytes if kind == "layer" else binding.decode_workspace_bytes
        s["ws_bytes"] = size(x.shape, x.w)
        s["ws"] = torch.empty(s["ws_bytes"], dtype=torch.uint8, device="cuda")
    return s


def run(s):
    x, kind = s["x"], s["kind"]
    if kind == "attention":
        binding.attention(s["q"], s["k"], s["v"], x.off_d, x.off_h, x.shape, 0.0, s["out"], s["lse"], s["tile_map"])
        return dict(out=s["out"], lse=s["lse"])
    if kind == "score":
        binding.score(s["q"], s["k"], s["lse"], x.off_d, x.off_h, x.shape, x.w, 0.0, s["scores"])
        return dict(scores=s["scores"])
    if kind == "select":
        binding.select(s["scores"], x.off_d, x.off_h, x.keep_d, x.keep_h, x.n, x.w, s["kept"], s["out_off"])
        binding.compact2(s["k"], s["k_out"], s["v"], s["v_out"], x.hkv * x.d * 2, s["kept"], x.kept)
    elif kind == "decode":
        binding.decode_update(s["q"], s["k"], s["v"], x.off_d, x.off_h, x.shape, x.w, 0.0, x.keep_d, x.keep_h, s["rw"], s["pos"],
                              s["scores"], s["kept"], s["out_off"], s["k_out"], s["v_out"], s["pos_out"], s["ws"], s["ws_bytes"])
    elif s["hidden"] is not None:
        binding.prefill_layer_fused(s["q"], s["k"], s["v"], x.off_d, x.off_h, x.shape, x.w, 0.0, x.keep_d, x.keep_h, s["rw"],
                                    s["hidden"], s["hidden"].shape[1] * 2, s["pos"], s["out"], s["scores"], s["kept"], s["out_off"],
                                    s["k_out"], s["v_out"], s["hidden_out"], s["pos_out"], s["ws"], s["ws_bytes"])
    elif s["rw"] is not None or s["pos"] is not None:
        binding.prefill_layer_ex(s["q"], s["k"], s["v"], x.off_d, x.off_h, x.shape, x.w, 0.0, x.keep_d, x.keep_h, s["rw"], s["pos"],
                                 s["out"], s["scores"], s["kept"], s["out_off"], s["k_out"], s["v_out"], s["pos_out"], s["ws"],
                                 s["ws_bytes"])
    else:
        binding.prefill_layer(s["q"], s["k"], s["v"], x.off_d, x.off_h, x.shape, x.w, 0.0, x.keep_d, x.keep_h, s["out"], s["scores"],
                              s["kept"], s["out_off"], s["k_out"], s["v_out"], s["ws"], s["ws_bytes"])
    r = dict(kept_idx=s["kept"], out_offsets=s["out_off"], k=s["k_out"].view(torch.int16), v=s["v_out"].view(torch.int16))
    if kind != "select":
        r["scores"] = s["scores"]
    if kind == "layer":
        r["out"] = s["out"]
    if s["hidden"] is not None:
        r["hidden"] = s["hidden_out"].view(torch.int16)
    if s["pos"] is not None:
        r["pos"] = s["pos_out"]
    return r


def work(case):
    lens = _lengths(case)
    T, kept = sum(lens), sum(_keeps(case, lens))
    hq, hkv, d, w, kind = case["hq"], case["hkv"], case["d"], case["w"], case["kind"]
    rows_q, rows_kv = 2 * hq * d, 2 * hkv * d
    causal = sum(2.0 * d * S * (S + 1) * hq for S in lens)                  # QK^T and PV under the diagonal
    strip = sum(2.0 * d * min(w, S) * S * hq for S in lens)                 # QK^T of the recent window
    gather = kept * (4 + (8 if case.get("pos") else 0) + (4 * case["hidden"] if case.get("hidden") else 0))
    win = sum(min(w, S) for S in lens)
    if kind == "attention":
        return dict(bytes=2 * T * (rows_q + rows_kv) + 4 * T * hq, flops=causal)
    if kind == "score":
        return dict(bytes=win * (rows_q + 4 * hq) + T * (rows_kv + 4), flops=strip)
    if kind == "select":
        return dict(bytes=4 * T + kept * (4 + 4 * rows_kv), flops=0)
    if kind == "decode":        # K in full, the kept rows of V, the kept rows out
        return dict(bytes=win * rows_q + T * (rows_kv + 4) + kept * 3 * rows_kv + gather, flops=strip)
    return dict(bytes=2 * T * (rows_q + rows_kv) + 4 * T + kept * 2 * rows_kv + gather, flops=causal)


def tolerance(case):
    kind = case["kind"]
    if kind == "select":
        return "exact"
    # Two correct selections may differ where two scores are equal to rounding; from the first such place on the ascending
    # list is shifted.  Measured against 64 bits over the listed cases: bf16 outputs rel 2.2e-3 and at most 6.4e-2 of the
    # rms (early rows are much larger than the mean over 32k keys), fp32 scores rel 3.6e-7 and at most 8.3e-7.
    if kind in ("layer", "attention"):
        return dict(rel=8e-3, max=0.25, differ=0.01)
    return dict(rel=1.5e-6, max=4e-6, differ=0.01)


def _window_logits(q, k, x):
    """[hq, L, S] logits of the last L positions against all S keys, masked; q [L, hq, d], k [S, hkv, d]."""
    L, S, g = q.shape[0], k.shape[0], x.hq // x.hkv
    qh = q.reshape(L, x.hkv, g, x.d).permute(1, 2, 0, 3).reshape(x.hkv, g * L, x.d).contiguous()
    kt = k.permute(1, 2, 0).contiguous()
    logits = torch.bmm(qh, kt).reshape(x.hq, L, S) * _scale(x.d)
    pos = torch.arange(S, device=q.device)
    return logits.masked_fill_((pos[None, :] > pos[S - L:, None])[None], -math.inf)


def _exact_scores(s, x, b):
    r0, r1 = x.off[b], x.off[b + 1]
    S = r1 - r0
    L = min(x.w, S)
    q = s["q"][b, x.w - L:] if s["kind"] == "decode" else s["q"][r1 - L:r1]
    logits = _window_logits(q.double(), s["k"][r0:r1].double(), x)
    if s["kind"] == "score":
        p = torch.exp(logits - s["lse"][r1 - L:r1].double().t()[:, :, None] * math.log(2.0))
    else:
        p = torch.softmax(logits, dim=2)
    wt = torch.ones(L, dtype=torch.float64, device="cuda") if s["rw"] is None else s["rw"][x.w - L:].double()
    return (p * wt[None, :, None]).sum(dim=(0, 1)) / (x.hq * wt.sum())


def _exact_attention(s, x, b, out, lse):
    r0, S, g = x.off[b], x.lens[b], x.hq // x.hkv
    kt = s["k"][r0:r0 + S].double().permute(1, 2, 0).contiguous()                       # [hkv, d, S]
    v = s["v"][r0:r0 + S].double().permute(1, 0, 2).contiguous()                        # [hkv, S, d]
    step = max(1, min(S, (1 << 27) // (x.hq * S)))
    for i in range(0, S, step):
        j = min(S, i + step)
        q = s["q"][r0 + i:r0 + j].double().reshape(j - i, x.hkv, g, x.d).permute(1, 2, 0, 3).reshape(x.hkv, g * (j - i), x.d)
        p = torch.bmm(q.contiguous(), kt[:, :, :j].contiguous()).mul_(_scale(x.d)).reshape(x.hkv, g, j - i, j)
        if i == 0 or j - i > 1:
            p.masked_fill_(torch.arange(j, device="cuda")[None, :] > torch.arange(i, j, device="cuda")[:, None], -math.inf)
        top = p.amax(dim=3, keepdim=True)
        p.sub_(top).exp_()
        den = p.sum(dim=3, keepdim=True)
        o = torch.bmm(p.reshape(x.hkv, g * (j - i), j), v[:, :j].contiguous()).reshape(x.hkv, g, j - i, x.d) / den
        out[r0 + i:r0 + j] = o.permute(2, 0, 1, 3).reshape(j - i, x.hq, x.d)
        if lse is not None:
            lse[r0 + i:r0 + j] = ((top + den.log())[..., 0] / math.log(2.0)).permute(2, 0, 1).reshape(j - i, x.hq)


def exact(case, seed):
    kind = case["kind"]
    if kind == "select":
        return None
    s = prepare(case, seed)
    x = s["x"]
    r = {}
    if kind in ("layer", "attention"):
        r["out"] = torch.empty(x.T, x.hq, x.d, dtype=torch.float64, device="cuda")
        if kind == "attention":
            r["lse"] = torch.empty(x.T, x.hq, dtype=torch.float64, device="cuda")
        for b in range(x.n):
            _exact_attention(s, x, b, r["out"], r.get("lse"))
    if kind != "attention":
        r["scores"] = torch.empty(x.T, dtype=torch.float64, device="cuda")
        for b in range(x.n):
            r["scores"][x.off[b]:x.off[b + 1]] = _exact_scores(s, x, b)
    if kind in ("layer", "decode"):                             # (whole numbers and copied bytes: nothing to round)
        r.update(kept_idx=None, out_offsets=None, k=None, v=None)
    return r
