"""The calls this library is timed with: what a program that trains or serves Parallel Evoformer blocks has it do.

A case names one call pattern (`call`), the block's sizes and widths, the storage type, the block ordering and the
number of streams:

  serve      pe_block_fwd_static: a forward pass without a workspace of the caller's (small blocks)
  infer      pe_block_fwd without saved activations
  train      d_params cleared, pe_block_fwd (activations saved), pe_block_bwd
  recompute  the same without saved activations between the two calls: the backward pass recomputes the forward
  trunk      d_params cleared, pe_stack_fwd_bwd over extra-MSA and main blocks

Channel widths are the three sets of pe_inputs.CONFIGS: "small" (its fp32 test block), "main" (Evoformer blocks) and
"extra" (extra-MSA blocks, global column attention).  Sequence and residue counts run from that configuration's
smallest block to its largest (s 8..5120, r 16..384).
"""
import math

import torch

import paper_2211_00235_amd as pe
from pe_inputs import dims_for

_WIDTHS = {"small": "tiny", "main": "af2_initial", "extra": "extra_msa"}
# largest estimated cost of a drawn case, in flops of the bf16 path; train_extra_msa_finetune is at 6.8e12
_MOST = 6e12
# pe_set_option number of "keep every block's activations" (PE_OPT_STACK_KEEP_CTX of include/pe.h)
_STACK_KEEP_CTX = 5


def _case(name, call, widths, s, r, dtype="bf16", ordering=0, streams=2, n_extra=0, n_main=0, s_extra=0, keep=False):
    c = dict(call=call, widths=widths, s=s, r=r, dtype=dtype, ordering=ordering, streams=streams, n_extra=n_extra,
             n_main=n_main, s_extra=s_extra, keep=keep)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest calls: launches and host work count.  A serving loop's forward pass on the library's own scratch ...
        _case("serve_small_fp32", "serve", "small", 24, 48, "fp32", streams=1),
        # ... and a training step of the smallest configured block
        _case("train_tiny_fp32", "train", "small", 8, 16, "fp32"),
        # inference on a short protein, whose length is what it is; one stream, as a plain PyTorch program has it
        _case("infer_short", "infer", "main", 128, 97, streams=1),
        # the block of AlphaFold2's initial training
        _case("train_initial", "train", "main", 128, 256),
        # a training crop of a protein shorter than the crop size, with fewer sequences than the cap: odd in both axes
        _case("train_ragged", "train", "main", 121, 237),
        # initial training in full precision
        _case("train_initial_fp32", "train", "main", 128, 256, "fp32"),
        # initial training of the AlphaFold2 ordering (outer product mean first, pair stack after it)
        _case("train_initial_af2", "train", "main", 128, 256, ordering=1),
        # extra-MSA block of initial training
        _case("train_extra_msa", "train", "extra", 1024, 256),
        # inference at the fine-tuning size
        _case("infer_finetune", "infer", "main", 512, 384),
        # fine-tuning with activations recomputed
        _case("recompute_finetune", "recompute", "main", 512, 384),
        # extra-MSA block of fine-tuning, the largest block there is
        _case("train_extra_msa_finetune", "train", "extra", 5120, 384),
        # a short trunk (the full one is 4 + 48 blocks of the same sizes), per-block recompute
        _case("trunk_short", "trunk", "main", 128, 256, n_extra=1, n_main=3, s_extra=1024),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        call = rng.choice(["serve", "infer", "infer", "train", "train", "train", "recompute", "trunk"])
        ordering = rng.choice([0, 0, 0, 1, 2])
        streams = rng.choice([1, 2, 2])
        if call == "serve":      # what fits the library's own scratch
            c = _case(None, call, "small", _log_int(rng, 8, 24), _log_int(rng, 16, 48), rng.choice(["fp32", "bf16"]),
                      ordering, streams)
        elif call == "trunk":
            c = _case(None, call, "main", _log_int(rng, 16, 160), _log_int(rng, 48, 256), "bf16", ordering, streams,
                      rng.choice([0, 1]), rng.choice([1, 2, 3]), _log_int(rng, 64, 1200), rng.random() < 0.5)
        else:
            w = rng.choice(["small", "main", "main", "main", "extra"])
            top = {"small": 64, "main": 512, "extra": 5120}[w]
            s = _log_int(rng, 8 if w == "small" else 16, top)
            r = _log_int(rng, 16, 64) if w == "small" else _log_int(rng, 33, 384)
            dtype = rng.choice(["fp32", "bf16"]) if w == "small" else rng.choice(["bf16", "bf16", "bf16", "fp32"])
            c = _case(None, call, w, s, r, dtype, ordering, streams)
        # fp32 contractions run at about a sixteenth of the bf16 rate
        if work(c)["flops"] * (16 if c["dtype"] == "fp32" else 1) <= _MOST:
            return c


def _dims(c, widths=None, s=None):
    d = dims_for(_WIDTHS[widths or c["widths"]])[0]
    d.update(s=s or c["s"], r=c["r"], dtype=pe.PE_F32 if c["dtype"] == "fp32" else pe.PE_BF16, variant=c["ordering"])
    return d


def _params(dims, n_blocks, gen):
    """LayerNorm gains near one, offsets and biases near zero, weights of variance 1 / fan_in: as after initialisation."""
    n = pe.param_count(dims)
    scale, shift = torch.empty(n), torch.zeros(n)
    for e in pe.param_table(dims):
        sl = slice(e["offset"], e["offset"] + math.prod(e["shape"]))
        scale[sl] = e["fan_in"] ** -0.5 if e["kind"] == "weight" else 0.1
        shift[sl] = 1.0 if e["kind"] == "ln_gamma" else 0.0
    p = torch.randn(n_blocks, n, generator=gen, device="cuda") * scale.cuda() + shift.cuda()
    return p.reshape(-1)


def _mask(n, share, gen):
    m = torch.ones(n, device="cuda")
    m[torch.randperm(n, generator=gen, device="cuda")[:int(round(share * n))]] = 0.0
    return m


_streams = []


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    d = _dims(case)
    s, r = d["s"], d["r"]
    dt = torch.float32 if case["dtype"] == "fp32" else torch.bfloat16

    def normal(*shape):
        return torch.randn(*shape, generator=gen, device="cuda", dtype=dt)

    st = {"call": case["call"], "dims": d, "h": pe.Handle()}
    st["msa"], st["pair"] = normal(s, r, d["c_m"]), normal(r, r, d["c_z"])
    if case["widths"] == "extra":           # 5 % of the sequences are padding
        st["msa_mask"] = _mask(s, 0.05, gen)[:, None].expand(s, r).contiguous()
        st["pair_mask"] = torch.ones(r, r, device="cuda")
    else:                                   # 10 % of the residues are unresolved
        m = _mask(r, 0.10, gen)
        st["msa_mask"], st["pair_mask"] = m[None, :].expand(s, r).contiguous(), (m[:, None] * m[None, :]).contiguous()
    blocks = case["n_main"] if case["call"] == "trunk" else 1
    st["params"] = _params(d, blocks, gen)
    st["msa_out"], st["pair_out"] = torch.empty_like(st["msa"]), torch.empty_like(st["pair"])
    if case["streams"] == 1:
        st["sm"] = st["sp"] = torch.cuda.current_stream()
    else:                                   # a program makes its two streams once
        while len(_streams) < 2:
            _streams.append(torch.cuda.Stream())
        st["sm"], st["sp"] = _streams
    byte = dict(dtype=torch.uint8, device="cuda")
    if case["call"] == "infer":
        st["ws"] = torch.empty(pe.workspace_bytes(d, 1), **byte)
    elif case["call"] in ("train", "recompute", "trunk"):
        st["d_msa_out"], st["d_pair_out"] = normal(s, r, d["c_m"]), normal(r, r, d["c_z"])
        st["d_msa_in"], st["d_pair_in"] = torch.empty_like(st["msa"]), torch.empty_like(st["pair"])
        st["ctx"] = torch.empty(pe.ctx_bytes(d), **byte) if case["call"] == "train" else None
        if case["call"] != "trunk":
            st["ws"] = torch.empty(pe.workspace_bytes(d, 0 if case["call"] == "train" else 1), **byte)
        else:
            st.update(n_extra=case["n_extra"], n_main=case["n_main"], de=None, ex=None, ex_mask=None, d_ex=None)
            if case["n_extra"]:
                e = st["de"] = _dims(case, "extra", case["s_extra"])
                st["ex"] = normal(e["s"], r, e["c_m"])
                st["ex_mask"] = _mask(e["s"], 0.05, gen)[:, None].expand(e["s"], r).contiguous()
                st["d_ex"] = torch.empty_like(st["ex"])
                st["params"] = torch.cat([_params(e, case["n_extra"], gen), st["params"]])
            if case["keep"]:
                st["h"].set_option(_STACK_KEEP_CTX, 1)
            st["ws"] = torch.empty(pe.stack_workspace_bytes(case["n_extra"], st["de"], case["n_main"], d,
                                                            keep=case["keep"]), **byte)
        st["d_params"] = torch.zeros_like(st["params"])
    return st


def run(st):
    x = (st["msa"], st["pair"], st["msa_mask"], st["pair_mask"], st["params"])
    out = [st["msa_out"], st["pair_out"]]
    if st["call"] == "serve":
        pe.block_fwd_static(st["h"], st["dims"], *x, *out, st["sm"], st["sp"])
        return out
    if st["call"] == "infer":
        pe.block_fwd(st["h"], st["dims"], *x, *out, None, st["ws"], st["sm"], st["sp"])
        return out
    with torch.cuda.stream(st["sm"]):
        st["d_params"].zero_()
    if st["call"] == "trunk":
        pe.stack_fwd_bwd(st["h"], st["n_extra"], st["de"], st["n_main"], st["dims"], st["ex"], st["msa"], st["pair"],
                         st["ex_mask"], st["msa_mask"], st["pair_mask"], st["params"], st["d_msa_out"], st["d_pair_out"],
                         *out, st["d_ex"], st["d_msa_in"], st["d_pair_in"], st["d_params"], st["ws"], st["sm"], st["sp"])
    else:
        pe.block_fwd(st["h"], st["dims"], *x, *out, st["ctx"], st["ws"], st["sm"], st["sp"])
        pe.block_bwd(st["h"], st["dims"], *x, st["d_msa_out"], st["d_pair_out"], st["d_msa_in"], st["d_pair_in"],
                     st["d_params"], st["ctx"], st["ws"], st["sm"], st["sp"])
    out += [st["d_msa_in"], st["d_pair_in"], st["d_params"]]
    if st["call"] == "trunk" and st["n_extra"]:
        out.append(st["d_ex"])
    return out


def _fwd_flops(d):
    """2 M N K per contraction of one block's forward pass, masked positions included."""
    s, r, cm, cz = d["s"], d["r"], d["c_m"], d["c_z"]
    mm, mz, hm, dm = s * r, r * r, d["h_msa"], d["d_msa"]
    hp, ct, co, n = d["h_pair"] * d["d_pair"], d["c_tri"], d["c_opm"], d["n_trans"]
    f = 10 * mm * cm * hm * dm + 2 * mz * cz * hm + 4 * s * r * r * hm * dm                  # row attention
    if d["col_global"]:
        f += 2 * mm * cm * (2 * hm * dm + 2 * dm) + 2 * r * cm * hm * dm + 4 * mm * hm * dm  # global column attention
    else:
        f += 10 * mm * cm * hm * dm + 4 * r * s * s * hm * dm                                # column attention
    f += 4 * n * mm * cm * cm                                                                # MSA transition
    f += 4 * mm * cm * co + 2 * (r * co) ** 2 * s + 2 * mz * co * co * cz                    # outer product mean
    f += 2 * (2 * mz * cz * (4 * ct + cz) + 2 * mz * ct * cz + 2 * r ** 3 * ct)              # triangle multiplications
    f += 2 * (10 * mz * cz * hp + 2 * mz * cz * d["h_pair"] + 4 * r ** 3 * hp)               # triangle attentions
    f += 4 * n * mz * cz * cz                                                                # pair transition
    return f


def work(case):
    """Each input read once, each output written once (cotangents and gradients of a training step among them);
    a training step is three times the forward's flops, recomputation is not counted."""
    d = _dims(case)
    b = 4 if case["dtype"] == "fp32" else 2
    grad = case["call"] in ("train", "recompute", "trunk")
    blocks = case["n_main"] if case["call"] == "trunk" else 1
    masks = 4 * (d["s"] * d["r"] + d["r"] * d["r"])
    act = b * (d["s"] * d["r"] * d["c_m"] + d["r"] * d["r"] * d["c_z"])
    par = 4 * blocks * pe.param_count(d)
    flops = blocks * _fwd_flops(d)
    if case["n_extra"]:
        e = _dims(case, "extra", case["s_extra"])
        masks += 4 * e["s"] * e["r"]
        act += b * e["s"] * e["r"] * e["c_m"] // 2      # read, and its cotangent written; there is no output
        par += 4 * case["n_extra"] * pe.param_count(e)
        flops += case["n_extra"] * _fwd_flops(e)
    return {"bytes": masks + (4 * act + 2 * par if grad else 2 * act + par), "flops": 3 * flops if grad else flops}


def tolerance(case):
    """Relative 2-norm error between two correct implementations.

    Forward: fp32 sums; in bf16 every intermediate tensor is rounded, the block's outputs are 6e-3 from float64
    (tests/test_gpu_stack.py), so 1e-2 between two paths.
    Backward: a hidden unit of a transition whose pre-activation is below its own rounding error may be on in one
    path and off in the other, and then its gradient differs by its whole size (tests/test_bf16_relu_band.py).
    bf16: 0.1 % of the units, which puts cotangents 3e-2 from float64.  fp32: about 5 of 33 million units
    (sqrt(5 / 16e6) of the active ones' norm, 6e-4), each of which moves one row."""
    grad = case["call"] in ("train", "recompute", "trunk")
    if case["dtype"] == "fp32":
        return {"rel": 1e-3, "max": 0.2} if grad else {"rel": 1e-5}
    return {"rel": 3e-2} if grad else {"rel": 1e-2}
