"""What users have this package do, as cases that can be timed and compared.

    layer     calibration statistics of one input, then one linear layer through the whole path
              (`activation_stats`, `quantize_layer` with the reconstruction error)
    block     a decoder block: statistics of every distinct input and all seven layers
              (`quantize_block`)
    retarget  a layer whose K-means runs per width are kept, at another average width
              (`quantize_layer_from_cache`)
    rtn       a layer through the uniform quantizer (`quantize_layer_rtn`)
    product   m tokens times the deployed layers that read the same input (`group_products`),
              the groups of a block one after the other

`listed()` names the cases, `draw()` gives more of the same ranges, `prepare()` / `run()` do the
work, `exact()` recomputes the floating-point outputs in 64 bits with plain torch.
"""
from __future__ import annotations

import math

import torch

from paper_2410_13056_amd import binding as B, pipeline as P, synth

DEV = "cuda"
_DTYPE = {"f16": torch.float16, "f32": torch.float32}


# ---------------------------------------------------------------------------------- cases

def _layer(name, d_out, d_in, tokens, dtype="f16", bits="234", avg=3.0, rho_q=5000, iters=20):
    return {"name": name, "kind": "layer", "d_out": d_out, "d_in": d_in, "tokens": tokens, "dtype": dtype,
            "bits": bits, "avg": avg, "rho_act": 4500, "rho_q": rho_q, "iters": iters}


def _product(name, shapes, m, bits="234", avg=3.5, rho_q=10000):
    """`shapes`: groups separated by '/', a group is d_in:d_out,d_out,..."""
    return {"name": name, "kind": "product", "shapes": shapes, "m": m, "bits": bits, "avg": avg,
            "rho_act": 4500, "rho_q": rho_q}


def listed():
    return [
        # the smallest configuration: an fp32 layer of a toy model, where launches and latency count
        _layer("layer_tiny_f32", 512, 256, 256, "f32", "23", 2.5, 5000, 10),
        # a key / value projection of the 70B-shaped block: many short channels
        _layer("layer_kv_1024x8192", 1024, 8192, 2048, avg=3.5, rho_q=10000),
        # an attention projection of a 7B-shaped model with its whole calibration set
        _layer("layer_4096x4096_262144tok", 4096, 4096, 262144),
        # sizes that are no multiple of anything (a pruned model, a resized vocabulary slice)
        _layer("layer_ragged_4099x3001", 4099, 3001, 1031),
        # a 7B-shaped block the way quantize_block runs by default: one stream
        {"name": "block_7b_one_stream", "kind": "block", "hidden": 4096, "ffn": 11008, "kv": 4096,
         "tokens": 65536, "bits": "23", "avg": 2.2, "rho_act": 4500, "rho_q": 500, "iters": 20, "streams": 1},
        # the 70B-shaped block of the benchmark, three streams: the largest call
        {"name": "block_70b_three_streams", "kind": "block", "hidden": 8192, "ffn": 28672, "kv": 1024,
         "tokens": 32768, "bits": "234", "avg": 3.5, "rho_act": 4500, "rho_q": 10000, "iters": 20, "streams": 3},
        # another deployment budget for the up projection of a 13B-shaped block
        {"name": "retarget_13824x5120", "kind": "retarget", "d_out": 13824, "d_in": 5120, "dtype": "f16",
         "bits": "234", "avg": 2.6, "rho_act": 4500, "rho_q": 5000, "iters": 20},
        # the uniform-quantizer variant on the same layer
        {"name": "rtn_13824x5120", "kind": "rtn", "d_out": 13824, "d_in": 5120, "dtype": "f16", "bits": "234",
         "avg": 3.5, "rho_act": 5000, "group": 128},
        # decode: one token through the products of the 70B-shaped block, launched as a decoder can
        # (query/key/value together, gate/up together)
        _product("decode_70b_1tok", "8192:8192,1024,1024/8192:8192/8192:28672,28672/28672:8192", 1),
        # decode of 16 sequences at once through the MLP input projections of a 13B-shaped block
        _product("decode_13b_mlp_16tok", "5120:13824,13824", 16, avg=2.5, rho_q=5000),
        # prefill: a prompt of 512 tokens through one attention and one MLP group of a 7B-shaped block
        _product("prefill_7b_512tok", "4096:4096,4096,4096/4096:11008,11008", 512, "23", 2.2, 500),
        # odd sizes and an odd number of tokens
        _product("product_ragged_5tok", "3001:4099,513", 5, "234", 3.0, 5000),
    ]


def _size(rng, lo, hi):
    """Log-uniform; four in ten are taken as drawn, the others are whole multiples of 64 (8 when small)."""
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if rng.random() < 0.4:
        return v
    step = 64 if v >= 256 else 8
    return max(step, v // step * step)


def _budget(rng):
    bits = rng.choice(["23", "234", "234", "34"])
    lo, hi = int(bits[0]), int(bits[-1])
    return bits, round(rng.uniform(lo, hi), 2)


def draw(rng):
    kind = rng.choices(["layer", "block", "retarget", "rtn", "product"], [4, 1, 1, 1, 5])[0]
    bits, avg = _budget(rng)
    rho_q = rng.choice([500, 5000, 10000])
    if kind == "layer":
        f32 = rng.random() < 0.15
        d_out = _size(rng, 64, 4096 if f32 else 16384)
        d_in = _size(rng, 64, 512 if f32 else 8192)
        c = _layer("", d_out, d_in, _size(rng, 64, 32768), "f32" if f32 else "f16", bits, avg, rho_q)
        del c["name"]
        return c
    if kind == "block":
        hidden = 8 * max(8, _size(rng, 32, 512))
        kv = hidden // rng.choice([1, 4, 8]) // 4 * 4
        return {"kind": "block", "hidden": hidden, "ffn": 4 * _size(rng, hidden // 4, hidden), "kv": kv,
                "tokens": _size(rng, 512, 32768), "bits": bits, "avg": avg, "rho_act": 4500, "rho_q": rho_q,
                "iters": 20, "streams": rng.choice([1, 3])}
    if kind == "retarget":
        return {"kind": "retarget", "d_out": _size(rng, 256, 16384), "d_in": _size(rng, 256, 8192), "dtype": "f16",
                "bits": bits, "avg": avg, "rho_act": 4500, "rho_q": rho_q, "iters": 20}
    if kind == "rtn":
        return {"kind": "rtn", "d_out": _size(rng, 256, 28672), "d_in": _size(rng, 256, 8192), "dtype": "f16",
                "bits": bits, "avg": avg, "rho_act": 5000, "group": rng.choice([64, 128])}
    m = rng.choice([1, 1, 1, 2, 4, 8]) if rng.random() < 0.5 else _size(rng, 9, 512)
    outs = [_size(rng, 64, 16384) for _ in range(rng.choice([1, 2, 3]))]
    c = _product("", f"{_size(rng, 256, 8192)}:{','.join(map(str, outs))}", m, bits, avg, rho_q)
    del c["name"]
    return c


# --------------------------------------------------------------------------------- inputs

def _bit_set(case):
    return tuple(int(b) for b in case["bits"])


def _layers_of_block(case):
    h, f, kv = case["hidden"], case["ffn"], case["kv"]
    return [("q_proj", h, h, "attn_in"), ("k_proj", kv, h, "attn_in"), ("v_proj", kv, h, "attn_in"),
            ("o_proj", h, h, "o_in"), ("gate_proj", f, h, "mlp_in"), ("up_proj", f, h, "mlp_in"),
            ("down_proj", h, f, "down_in")]


def _statistic(d_in, seed):
    """A channel statistic as calibration leaves it: a log-normal spread and a few hot channels."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    s = torch.exp(torch.randn(d_in, generator=g, device=DEV))
    hot = torch.randperm(d_in, generator=g, device=DEV)[:max(1, d_in // 100)]
    s[hot] *= 900.0
    return s * 1000.0


def _groups(case):
    """[(d_in, [d_out, ...]), ...] of a product case."""
    out = []
    for g in case["shapes"].split("/"):
        d_in, outs = g.split(":")
        out.append((int(d_in), [int(v) for v in outs.split(",")]))
    return out


def _count(ppm, n):
    return (2 * ppm * n + 1_000_000) // 2_000_000


def _widths(stat, case):
    """O_act, the width of every other channel (16 for O_act) and the channels per width: the k
    largest statistics are kept whole, then Algorithm 1 with an integer budget."""
    d_in, s = stat.numel(), _bit_set(case)
    k_act = _count(case["rho_act"], d_in)
    order = torch.sort(stat, descending=True, stable=True).indices
    d_eff, avg = d_in - k_act, case["avg"]
    rest = order[k_act:]
    lo = max(b for b in s if b <= avg)
    bits = torch.full((d_in,), 16, dtype=torch.uint8, device=stat.device)
    bits[rest] = lo
    if avg > lo:
        bits[rest[:int(math.floor(avg * d_eff + 1e-9)) - lo * d_eff]] = lo + 1
    elif lo - 1 in s and lo + 1 in s:
        n = math.ceil(0.01 * (d_eff - 1)) if d_eff > 0 else 0
        if n > 0:
            bits[rest[:n]] = lo + 1
            bits[rest[d_eff - n:]] = lo - 1
    return torch.sort(order[:k_act]).values, bits, [int((bits == b).sum()) for b in s]


_CHUNK = 1 << 26      # weights worked on at a time while inputs are made


class _Stored:
    """A deployed layer made directly in the stored format: levels at normal quantiles, codes of
    normal weights, O_q at random places with heavy-tailed values."""

    def __init__(self, case, d_in, d_out, stat, seed):
        self.d_in, self.d_out, self.seed, self.bit_set = d_in, d_out, seed, _bit_set(case)
        self.act_idx, self.bits, self.counts = _widths(stat, case)
        g = self._gen(1)
        self.chan = [torch.nonzero(self.bits == b).flatten() for b in self.bit_set]
        self.lut = []
        for b, rows in zip(self.bit_set, self.chan):
            p = (torch.arange(1 << b, device=DEV, dtype=torch.float32) + 0.5) / (1 << b)
            q = torch.special.ndtri(p) * 1.15
            scale = 0.02 * torch.exp(0.2 * torch.randn((rows.numel(), 1), generator=g, device=DEV))
            self.lut.append((q * scale).to(torch.float16))
        self.W_act = (0.02 * torch.randn((self.act_idx.numel(), d_out), generator=g, device=DEV)).to(torch.float16)
        n = _count(case["rho_q"], d_in * d_out)
        lin = torch.unique(torch.randint(0, d_in * d_out, (n,), generator=g, device=DEV)) if n else \
            torch.empty(0, dtype=torch.int64, device=DEV)
        lin = lin[self.bits[lin // d_out] != 16]
        v = torch.randn(lin.numel(), generator=g, device=DEV)
        self.out_lin, self.out_val = lin, (torch.sign(v) * 0.06 + 0.03 * v).to(torch.float16)

    def _gen(self, j):
        return torch.Generator(device=DEV).manual_seed(self.seed * 97 + j)

    def codes(self):
        """(width position, first row, codes) in chunks of rows, the same on every call."""
        for j, (b, rows) in enumerate(zip(self.bit_set, self.chan)):
            g = self._gen(10 + j)
            step = max(1, _CHUNK // self.d_out)
            p = torch.arange(1, 1 << b, device=DEV, dtype=torch.float32) / (1 << b)
            for r0 in range(0, rows.numel(), step):
                n = min(step, rows.numel() - r0)
                u = torch.rand((n, self.d_out), generator=g, device=DEV)
                yield j, r0, torch.bucketize(u, p).to(torch.uint8)

    def dense(self):
        """(channels, W_hat rows in 64 bits) in chunks."""
        for j, r0, c in self.codes():
            ch = self.chan[j][r0:r0 + c.shape[0]]
            w = torch.gather(self.lut[j][r0:r0 + c.shape[0]].double(), 1, c.long())
            row_of = torch.full((self.d_in,), -1, dtype=torch.int64, device=DEV)
            row_of[ch] = torch.arange(ch.numel(), device=DEV)
            r = row_of[self.out_lin // self.d_out]
            hit = r >= 0
            w[r[hit], (self.out_lin % self.d_out)[hit]] = self.out_val[hit].double()
            yield ch, w
        if self.act_idx.numel():
            yield self.act_idx, self.W_act.double()

    def deployed(self):
        d_in, d_out = self.d_in, self.d_out
        packed = [torch.empty((r.numel(), (d_out * b + 31) // 32), dtype=torch.int32, device=DEV)
                  for b, r in zip(self.bit_set, self.chan)]
        level = torch.empty(self.out_lin.numel(), dtype=torch.float32, device=DEV)
        out_row = self.out_lin // d_out
        for j, r0, c in self.codes():
            n = c.shape[0]
            packed[j][r0:r0 + n] = _pack(c, self.bit_set[j])
            row_of = torch.full((d_in,), -1, dtype=torch.int64, device=DEV)
            row_of[self.chan[j][r0:r0 + n]] = torch.arange(n, device=DEV)
            r = row_of[out_row]
            hit = torch.nonzero(r >= 0).flatten()
            code = c[r[hit], (self.out_lin % d_out)[hit]].long()
            level[hit] = self.lut[j][r0:r0 + n][r[hit], code].float()
        col = self.out_lin % d_out
        by_col = torch.argsort(col * d_in + out_row)
        colptr = torch.zeros(d_out + 1, dtype=torch.int32, device=DEV)
        colptr[1:] = torch.cumsum(torch.bincount(col, minlength=d_out), 0)
        some = lambda ts: [t if t.shape[0] else None for t in ts]  # noqa: E731
        return P.Deployed(d_in, d_out, self.bit_set, self.counts, some(packed),
                          some([r.to(torch.int32) for r in self.chan]), some(self.lut),
                          self.act_idx.to(torch.int32), self.W_act, colptr, out_row[by_col].to(torch.int32),
                          (self.out_val.float() - level)[by_col])


def _pack(codes, b):
    """A little-endian bit stream per row, padded to whole 32-bit words."""
    rows, d_out = codes.shape
    pad = -d_out % 32
    c = torch.nn.functional.pad(codes, (0, pad)).to(torch.int64) if pad else codes.to(torch.int64)
    bits = b
    for _ in range(4):                                      # 16 codes to one 64-bit word
        c = c[:, 0::2] | (c[:, 1::2] << bits)
        bits *= 2
    lo, hi = c[:, 0::2], c[:, 1::2]
    mask = 0xffffffff
    if b == 4:
        words = [lo & mask, (lo >> 32) & mask, hi & mask, (hi >> 32) & mask]
    elif b == 3:
        words = [lo & mask, (lo >> 32) | ((hi & 0xffff) << 16), hi >> 16]
    elif b == 2:
        words = [lo, hi]
    else:
        words = [lo | (hi << 16)]
    w = torch.stack(words, 2).reshape(rows, -1)[:, :(d_out * b + 31) // 32]
    return torch.where(w >= 1 << 31, w - (1 << 32), w).to(torch.int32)


def _products(case, seed):
    """[(X, [_Stored, ...])] of a product case."""
    out = []
    for gi, (d_in, outs) in enumerate(_groups(case)):
        X = synth.make_activations(case["m"], d_in, "f16", seed * 1000 + gi, DEV)
        stat = _statistic(d_in, seed * 1000 + 100 + gi)
        out.append((X, [_Stored(case, d_in, o, stat, seed * 1000 + 200 + 10 * gi + li) for li, o in enumerate(outs)]))
    return out


def prepare(case, seed):
    kind = case["kind"]
    st = {"case": case}
    if kind == "layer":
        st["W"] = synth.make_weight(case["d_out"], case["d_in"], case["dtype"], seed * 1000, DEV)
        st["X"] = synth.make_activations(case["tokens"], case["d_in"], case["dtype"], seed * 1000 + 1, DEV)
        st["ws"] = B.Workspace(DEV)
    elif kind == "block":
        st["weights"], st["acts"] = {}, {}
        for j, (name, d_out, d_in, key) in enumerate(_layers_of_block(case)):
            st["weights"][name] = synth.make_weight(d_out, d_in, "f16", seed * 1000 + j, DEV)
            if key not in st["acts"]:
                st["acts"][key] = synth.make_activations(case["tokens"], d_in, "f16", seed * 1000 + 100 + j, DEV,
                                                         gated=key == "down_in")
        n = case["streams"]
        st["ws"] = B.Workspace(DEV) if n == 1 else [B.Workspace(DEV) for _ in range(n)]
    elif kind in ("retarget", "rtn"):
        W = synth.make_weight(case["d_in"], case["d_out"], case["dtype"], seed * 1000, DEV)    # already [d_in, d_out]
        st["sumsq"], st["ws"] = _statistic(case["d_in"], seed * 1000 + 1), B.Workspace(DEV)
        if kind == "rtn":
            st["W"] = W
        else:
            st["cache"] = P.build_width_cache(W, _bit_set(case), case["iters"], st["ws"], transposed=True)
    else:
        st["ws"], st["groups"] = B.Workspace(DEV), []
        for X, layers in _products(case, seed):
            deps = [s.deployed() for s in layers]
            Ys = [torch.empty((case["m"], d.d_out), dtype=torch.float32, device=DEV) for d in deps]
            st["groups"].append((P.group_products(deps), [X] * len(deps), Ys))
    return st


# ------------------------------------------------------------------------------------ run

def _outputs(r, codes=True):
    out = {"bits": r.bits, "centroids": r.centroids, "out_idx": r.out_idx, "out_val": r.out_val,
           "packed": r.packed, "err_ch": r.err_ch, "err_total": r.err_total}
    if codes:
        out.update(codes=r.codes, chan_idx=r.chan_idx, lut=r.lut, sumsq=r.sumsq, act_idx=r.act_idx)
    return out


def run(st):
    case, kind = st["case"], st["case"]["kind"]
    if kind == "layer":
        sumsq = P.activation_stats(st["X"], st["ws"])[1]
        return _outputs(P.quantize_layer(st["W"], sumsq, _bit_set(case), case["avg"], case["rho_act"], case["rho_q"],
                                         case["iters"], st["ws"], with_error=True))
    if kind == "block":
        out = P.quantize_block(st["weights"], st["acts"], [(n, k) for n, _, _, k in _layers_of_block(case)],
                               _bit_set(case), case["avg"], case["rho_act"], case["rho_q"], case["iters"], st["ws"],
                               with_error=True, streams=case["streams"])
        return {n: _outputs(r, codes=False) for n, r in out.items()}      # the codes are in the packed rows
    if kind == "retarget":
        return _outputs(P.quantize_layer_from_cache(st["cache"], st["sumsq"], case["avg"], case["rho_act"],
                                                    case["rho_q"], st["ws"], with_error=True))
    if kind == "rtn":
        r = P.quantize_layer_rtn(st["W"], st["sumsq"], _bit_set(case), case["avg"], case["rho_act"], case["group"],
                                 st["ws"], with_error=True, transposed=True)
        return {"bits": r.bits, "codes": r.codes, "scale": r.scale, "zero": r.zero, "err_ch": r.err_ch}
    for call, xs, ys in st["groups"]:
        call(xs, ys, st["ws"])
    return [ys for _, _, ys in st["groups"]]


# ----------------------------------------------------------------------------------- work

def _stored_bytes(d_in, d_out, avg):
    return d_in * d_out * avg / 8 + d_in * (2 * 2 ** avg + 4)


def _quantize_work(d_in, d_out, case, esz):
    n_q = _count(case["rho_q"], d_in * d_out)
    return {"bytes": d_in * d_out * (esz + 1) + _stored_bytes(d_in, d_out, case["avg"]) + n_q * 6 + d_in * 80,
            # per weight and pass: found and added once (the rounds can work on sums), coded once
            "flops": 8 * d_in * d_out}


def work(case):
    kind = case["kind"]
    if kind == "layer":
        esz = _DTYPE[case["dtype"]].itemsize
        w = _quantize_work(case["d_in"], case["d_out"], case, esz)
        n = case["tokens"] * case["d_in"]
        return {"bytes": w["bytes"] + n * esz, "flops": w["flops"] + 2 * n}
    if kind == "block":
        w, keys = {"bytes": 0, "flops": 0}, set()
        for _, d_out, d_in, key in _layers_of_block(case):
            q = _quantize_work(d_in, d_out, case, 2)
            n = 0 if key in keys else case["tokens"] * d_in
            keys.add(key)
            w["bytes"] += q["bytes"] + 2 * n
            w["flops"] += q["flops"] + 2 * n
        return w
    if kind == "retarget":                       # the kept run's codes stand in for the first pass
        w = _quantize_work(case["d_in"], case["d_out"], case, 2)
        return {"bytes": w["bytes"] + case["d_in"] * case["d_out"], "flops": w["flops"]}
    if kind == "rtn":
        n = case["d_in"] * case["d_out"]
        return {"bytes": 3 * n + 8 * n / case["group"], "flops": 6 * n}
    w = {"bytes": 0, "flops": 0}
    for d_in, outs in _groups(case):
        w["bytes"] += 2 * case["m"] * d_in
        for d_out in outs:
            w["bytes"] += _stored_bytes(d_in, d_out, case["avg"]) + 4 * case["m"] * d_out + 4 * d_out \
                + _count(case["rho_act"], d_in) * 2 * d_out + _count(case["rho_q"], d_in * d_out) * 8
            w["flops"] += 2 * case["m"] * d_in * d_out
    return w


def tolerance(case):
    # Products: fp32 sums of up to 28672 terms, measured 1.1e-7 to 1.5e-7 off the exact ones.
    # Everything else is fp64 (or whole numbers) rounded once to fp32: an ulp where the order of
    # the fp64 sums tips the rounding.
    return {"rel": 6e-7} if case["kind"] == "product" else {"rel": 1.2e-7}


# ---------------------------------------------------------------------------- in 64 bits

def _lloyd(V, keep, K, iters):
    """Levels [c, K] fp32 of channels V [c, n] (fp64) without the entries where keep is False."""
    n = V.shape[1]
    S = torch.where(keep, V, torch.inf) if keep is not None else V
    S = torch.sort(S, dim=1).values
    M = keep.sum(1) if keep is not None else torch.full((V.shape[0],), n, device=V.device)
    prefix = torch.nn.functional.pad(torch.cumsum(torch.where(torch.isfinite(S), S, 0.0), 1), (1, 0))
    j = torch.arange(K, device=V.device)
    start = torch.div((2 * j + 1)[None] * M[:, None], 2 * K, rounding_mode="floor").clamp(max=n - 1)
    levels = torch.gather(S, 1, start).float()
    edge0, edgeM = torch.zeros_like(M)[:, None], M[:, None]
    for _ in range(iters):
        mid = (levels[:, :-1].double() + levels[:, 1:].double()) / 2
        at = torch.cat([edge0, torch.minimum(torch.searchsorted(S, mid, right=True), edgeM), edgeM], 1)
        count = at[:, 1:] - at[:, :-1]
        total = torch.gather(prefix, 1, at[:, 1:]) - torch.gather(prefix, 1, at[:, :-1])
        levels = torch.where(count > 0, (total / count.clamp(min=1)).float(), levels)
    return levels


def _code(V, levels):
    """The nearest level of every weight, the lower one where two are as near."""
    mid = (levels[:, :-1].double() + levels[:, 1:].double()) / 2
    return torch.searchsorted(mid, V)


def _exact_layer(W, stat, case):
    """W [d_in, d_out]: levels, errors per channel and in total, in 64 bits."""
    d_in, d_out = W.shape
    V = W.double() + 0.0
    _, bits, _ = _widths(stat, case)
    score = torch.full((d_in, d_out), -1.0, dtype=torch.float32, device=W.device)
    rows = {b: torch.nonzero(bits == b).flatten() for b in _bit_set(case)}
    for b, r in rows.items():
        if r.numel():
            q = _lloyd(V[r], None, 1 << b, case["iters"])
            score[r] = (V[r] - torch.gather(q.double(), 1, _code(V[r], q))).abs().float()
    k = _count(case["rho_q"], d_in * d_out)
    keep = torch.ones(d_in * d_out, dtype=torch.bool, device=W.device)
    keep[torch.sort(score.flatten(), descending=True, stable=True).indices[:k]] = False
    keep = keep.view(d_in, d_out)
    cent = torch.full((d_in, 16), torch.inf, dtype=torch.float64, device=W.device)
    diff = W.double() - W.to(torch.float16).double()            # what is kept in FP16
    for b, r in rows.items():
        if r.numel():
            q = _lloyd(V[r], keep[r], 1 << b, case["iters"]).double()
            cent[r, :1 << b] = q
            diff[r] = torch.where(keep[r], V[r] - torch.gather(q, 1, _code(V[r], q.float())), diff[r])
    err = (diff * diff).sum(1)
    return {"centroids": cent, "err_ch": err, "err_total": torch.stack([(err * stat.double()).sum(), err.sum()])}


def exact(case, seed):
    kind = case["kind"]
    if kind == "layer":
        X = synth.make_activations(case["tokens"], case["d_in"], case["dtype"], seed * 1000 + 1, DEV)
        stat = sum((c.double() ** 2).sum(0) for c in X.split(8192))
        W = synth.make_weight(case["d_out"], case["d_in"], case["dtype"], seed * 1000, DEV).t().contiguous()
        return {**_exact_layer(W, stat.float(), case), "sumsq": stat}
    if kind == "block":
        return None
    if kind in ("retarget", "rtn"):
        W = synth.make_weight(case["d_in"], case["d_out"], case["dtype"], seed * 1000, DEV)
        stat = _statistic(case["d_in"], seed * 1000 + 1)
        if kind == "retarget":
            return {**_exact_layer(W, stat, case), "sumsq": stat.double()}
        g, V = case["group"], W.double()
        _, bits, _ = _widths(stat, case)
        pad = -V.shape[1] % g
        G = torch.nn.functional.pad(V, (0, pad), mode="replicate") if pad else V
        G = G.view(V.shape[0], -1, g)
        live = (bits != 16)[:, None]
        lo = G.amin(2)
        step = (G.amax(2) - lo) / ((1 << torch.where(live, bits[:, None], 1).long()) - 1)
        code = torch.round((G - lo[..., None]) / torch.where(step == 0, 1.0, step)[..., None])
        d = (G - (lo[..., None] + code * step[..., None])).view(V.shape[0], -1)[:, :V.shape[1]]
        return {"scale": torch.where(live, step, 0.0), "zero": torch.where(live, lo, 0.0),
                "err_ch": torch.where(live[:, 0], (d * d).sum(1), 0.0)}
    out = []
    for X, layers in _products(case, seed):
        ys = []
        for s in layers:
            y = torch.zeros((case["m"], s.d_out), dtype=torch.float64, device=DEV)
            for ch, w in s.dense():
                y += X[:, ch].double() @ w
            ys.append(y)
        out.append(ys)
    return out
