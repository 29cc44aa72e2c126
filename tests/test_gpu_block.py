"""GPU parity of pe_block_fwd / pe_block_bwd against the float64 oracle (through the C ABI)."""
import numpy as np
import pytest

import paper_2211_00235_amd as pe
from oracle import evoformer as ev
from oracle.params import param_table
from pe_inputs import make_inputs, dims_for
from tests.gpu_util import BlockRun, to_np, rel_err, param_errors
from tests.parity import TOL, check_case, relu_decisions, worst_scaled

pytestmark = pytest.mark.gpu


def _case(name, dtype=None, **over):
    dims, mask, seed = dims_for(name)
    dims.update(over)
    if dtype is not None:
        dims["dtype"] = dtype
    table, n = param_table(dims)
    return dims, table, make_inputs(dims, table, n, mask, seed)


def _assert(errs, worst, tol, stats):
    """Every tensor is held to the tolerance of the path times the size factor of the metric for its number of
    entries (tests/parity.py: SIZE_FACTORS; 1.0 above 4096 entries, so outputs, cotangents, saved activations and the
    larger weights are held to the plain tolerance): the metric divides by the tensor's largest reference magnitude,
    which for a tensor of a few hundred entries is a small-sample maximum."""
    worst, val = worst_scaled(errs, stats["sizes"])
    assert val <= tol, "worst %s = %.3e (after its size factor %.3e) > %.1e" % (worst, errs[worst], val, tol)


def test_tiny_fp32():
    """Config 1: tiny block, fp32 path, tolerance 1e-4."""
    dims, table, inp = _case("tiny")
    _assert(*check_case(dims, table, inp))


def _assert_small(errs, tol, stats):
    _assert(errs, None, tol, stats)


def test_tiny_bf16():
    dims, table, inp = _case("tiny", dtype=1)
    errs, worst, tol, stats = check_case(dims, table, inp)
    _assert_small(errs, tol, stats)


@pytest.mark.parametrize("dtype", [0, 1])
def test_ragged_shapes(dtype):
    """Sizes that are not multiples of any tile (s=37, r=150): several tiles plus ragged tails
    in every kernel; 11 masked residues."""
    dims, table, inp = _case("tiny", dtype=dtype, s=37, r=150, c_m=64, c_z=32, h_msa=2, d_msa=16, h_pair=4,
                             d_pair=8, c_tri=24, c_opm=16, n_trans=2)
    table, n = param_table(dims)
    inp = make_inputs(dims, table, n, ("random_residues", 0.07), 5)
    errs, worst, tol, stats = check_case(dims, table, inp)
    if dtype == 1:
        _assert_small(errs, tol, stats)
    else:
        _assert(errs, worst, tol, stats)


@pytest.mark.parametrize("dtype", [0, 1])
def test_head_dim_24(dtype):
    """Head dimension 24 (three 8-channel groups per head): the attention kernels pad the contraction, and the
    backward takes the separate pre-pass instead of the fused GEMM epilogue, which wants 8, 16 or 32."""
    dims, table, inp = _case("tiny", dtype=dtype, s=20, r=72, c_m=64, c_z=32, h_msa=2, d_msa=24, h_pair=2,
                             d_pair=24, c_tri=16, c_opm=8, n_trans=2)
    table, n = param_table(dims)
    inp = make_inputs(dims, table, n, ("random_residues", 0.1), 9)
    errs, worst, tol, stats = check_case(dims, table, inp)
    if dtype == 1:
        _assert_small(errs, tol, stats)
    else:
        _assert(errs, worst, tol, stats)


@pytest.mark.parametrize("c_tri,r", [(64, 36), (128, 20)])
def test_triangle_channel_major_layernorm_bf16(c_tri, r):
    """bf16 with 64 and 128 triangle channels and r * r a multiple of 8 but not of 128: the channel-major LayerNorm
    kernels that move 256-byte runs through a swizzled LDS tile (both lane-group widths), with a ragged last
    workgroup; the transition's ReLU decisions travel as bits (channel counts are multiples of 8)."""
    dims, table, inp = _case("tiny", dtype=1, s=12, r=r, c_m=32, c_z=32, h_msa=2, d_msa=16, h_pair=2, d_pair=16,
                             c_tri=c_tri, c_opm=8, n_trans=2)
    table, n = param_table(dims)
    inp = make_inputs(dims, table, n, ("random_residues", 0.1), 17)
    errs, worst, tol, stats = check_case(dims, table, inp)
    _assert_small(errs, tol, stats)


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("c_tri,r", [(32, 1), (32, 7), (64, 9), (128, 67), (96, 130), (32, 133)])
def test_triangle_planes_with_padded_pitch(c_tri, r, dtype):
    """Residue counts that are not multiples of 8: the channel-major planes get a row pitch of r rounded up to 8 with
    zeros in the padding.  One row short of a multiple, one row beyond one, more than one 128-row tile; channel counts
    of both channel-major LayerNorm kernels; nothing of the padding may reach an output or a gradient."""
    dims, table, inp = _case("tiny", dtype=dtype, s=5, r=r, c_tri=c_tri, c_z=32)
    table, n = param_table(dims)
    inp = make_inputs(dims, table, n, ("random_residues", 0.1), 23)
    errs, worst, tol, stats = check_case(dims, table, inp)
    _assert(errs, worst, tol, stats)


@pytest.mark.parametrize("c_tri,r", [(32, 2), (64, 3), (32, 4)])
def test_triangle_planes_at_the_smallest_residue_counts_fp32(c_tri, r):
    """Both sides of the rule for the pitch (r rounded up to 8 from r = 4 on).  fp32 only: over 4 or 9 pair positions the
    rounding errors of bf16 do not average out (its parameter gradients reach 3e-2 here, with and without padding);
    test_results_do_not_depend_on_what_the_buffers_held has the same sizes in bf16."""
    dims, table, inp = _case("tiny", s=5, r=r, c_tri=c_tri, c_z=32)
    table, n = param_table(dims)
    inp = make_inputs(dims, table, n, ("none", 0), 23)
    _assert(*check_case(dims, table, inp))


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("r", [1, 2, 3, 4, 5, 9, 20])
def test_results_do_not_depend_on_what_the_buffers_held(r, dtype):
    """The same call with ctx and workspace full of zeros and full of NaN (0xff bytes, in either type) before each pass:
    nothing that was not written may reach an output or a gradient, not even times zero.  Residue counts with and
    without padding in the channel-major planes, and the smallest, whose rows are followed by other tensors at once."""
    dims, table, inp = _case("tiny", dtype=dtype, s=5, r=r, c_tri=32, c_z=32)
    table, n = param_table(dims)
    inp = make_inputs(dims, table, n, ("none", 0), 31)
    got = []
    for fill in (0, 255):
        run = BlockRun(dims, inp)
        run.ctx.fill_(fill)
        run.ws.fill_(fill)
        run.sync()
        run.fwd(use_ctx=True)
        run.sync()
        run.ws.fill_(fill)
        run.sync()
        run.bwd(use_ctx=True)
        run.sync()
        got.append([to_np(t) for t in (run.msa_out, run.pair_out, run.d_msa_in, run.d_pair_in, run.d_params)])
    for a, b in zip(*got):
        assert np.isfinite(a).all() and np.array_equal(a, b)


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("s,r,c_m,c_z", [(1, 31, 32, 16), (33, 33, 24, 32), (7, 65, 64, 16), (3, 34, 128, 16)])
def test_small_problem_gemms(s, r, c_m, c_z, dtype):
    """The 32 x 32-tile GEMM kernel: row counts one short of and one beyond its tiles, unaligned contractions (odd r),
    channel counts at and beyond the limits of its LayerNorm prologue (64 fp32, 128 bf16) and of its LayerNorm-backward
    epilogue (32), a channel count that leaves half a k-chunk (24), a half-empty column tile.  (Not fewer than 16 pair channels: the bf16
    pre-activation bound of tests/parity.py was measured from 32 channels up, and the error of a LayerNorm over n channels
    relative to its own spread grows like n^-1/2: 8 channels reach 4.9e-2 against its 4e-2.)"""
    dims, table, inp = _case("tiny", dtype=dtype, s=s, r=r, c_m=c_m, c_z=c_z)
    table, n = param_table(dims)
    inp = make_inputs(dims, table, n, ("random_residues", 0.1), 29)
    names = _kernel_launches(BlockRun(dims, inp))
    for form in ("kc,kc", "LayerNorm", "EpiLnBwd"):
        assert names.get("gemm_small_kernel<%s>" % form, 0) > 0, (form, names)
    errs, worst, tol, stats = check_case(dims, table, inp)
    _assert(errs, worst, tol, stats)


@pytest.mark.parametrize("use_ctx", [True, False])
@pytest.mark.parametrize("dtype,r", [(0, 19), (1, 19), (1, 40), (0, 32), (1, 32)])
def test_row_complete_layernorm_epilogues(dtype, r, use_ctx):
    """128 pair channels: the pair stack's output projections write the next sub-operation's LayerNorm and its
    cotangent GEMMs finish the LayerNorm backward on their 64 x 128 tiles.  r * r = 361 leaves a ragged last tile of
    41 rows (and rows beyond the matrix in both 32-row halves); r * r = 1600 is made of full tiles; with r = 32 (a
    multiple of the attention kernels' 32-position tiles) no tile of the bias gradient is padded; the fused backward
    epilogue gathers that gradient from the tiled sum at every r.  With and without a saved ctx (the recomputed forward
    takes the same kernels)."""
    dims, table, inp = _case("tiny", dtype=dtype, s=9, r=r, c_m=32, c_z=128, h_msa=2, d_msa=16, h_pair=4, d_pair=32,
                             c_tri=32, c_opm=8, n_trans=2)
    table, n = param_table(dims)
    inp = make_inputs(dims, table, n, ("random_residues", 0.1), 23)
    errs, worst, tol, stats = check_case(dims, table, inp, use_ctx=use_ctx)
    if dtype == 1:
        _assert_small(errs, tol, stats)
    else:
        _assert(errs, worst, tol, stats)


@pytest.mark.parametrize("dtype", [0, 1])
def test_row_complete_layernorm_epilogues_eight_pair_heads(dtype):
    """The same with eight pair heads: the bias path of the fused epilogues is built for up to four and for up to
    eight heads."""
    dims, table, inp = _case("tiny", dtype=dtype, s=6, r=24, c_m=32, c_z=128, h_msa=2, d_msa=16, h_pair=8, d_pair=16,
                             c_tri=32, c_opm=8, n_trans=2)
    table, n = param_table(dims)
    inp = make_inputs(dims, table, n, ("random_residues", 0.1), 31)
    errs, worst, tol, stats = check_case(dims, table, inp)
    if dtype == 1:
        _assert_small(errs, tol, stats)
    else:
        _assert(errs, worst, tol, stats)


@pytest.mark.parametrize("c_z", [16, 128])
def test_single_branch_option_matches_the_full_block(c_z):
    """PE_OPT_BRANCHES: a call that runs one branch only leaves that branch's saved activations and input cotangent as
    the full block computes them (Section "Parallel Evoformer": the branches are independent inside a block).  fp32;
    c_z = 128 takes the fused epilogues, whose last launch adds the MSA branch's term only when that branch runs.
    Pair branch alone: z1..z5 bit-identical to the full block's; d_pair_in = the full block's d_pair_in minus the
    row-attention-bias term, which the MSA branch alone delivers as its d_pair_in."""
    import torch
    import paper_2211_00235_amd as pe
    from paper_2211_00235_amd.harness import BlockRun
    dims, table, inp = _case("tiny", dtype=0, s=7, r=24, c_m=32, c_z=c_z, h_msa=2, d_msa=16, h_pair=2, d_pair=16, c_tri=16,
                             c_opm=8, n_trans=2)
    table, n = param_table(dims)
    inp = make_inputs(dims, table, n, ("random_residues", 0.1), 37)
    runs = {}
    for br in (3, 2, 1):
        run = BlockRun(dims, inp)
        run.h.set_option(1, br)   # PE_OPT_BRANCHES
        run.d_pair_in.zero_()
        run.d_msa_in.zero_()
        run.fwd()
        run.bwd()
        run.sync()
        runs[br] = run
    full, pair_only, msa_only = runs[3], runs[2], runs[1]
    for k in ("z1", "z2", "z3", "z4", "z5"):
        assert np.array_equal(pair_only.ctx_entry(k), full.ctx_entry(k)), k
    for k in ("m1", "m2", "m3"):
        assert np.array_equal(msa_only.ctx_entry(k), full.ctx_entry(k)), k
    assert torch.equal(msa_only.d_msa_in, full.d_msa_in)
    dz_full = full.d_pair_in.double().cpu().numpy()
    dz_sum = pair_only.d_pair_in.double().cpu().numpy() + msa_only.d_pair_in.double().cpu().numpy()
    assert np.max(np.abs(dz_full - dz_sum)) <= 2e-6 * np.max(np.abs(dz_full))


@pytest.mark.parametrize("variant,use_ctx", [(0, True), (0, False), (2, True)])
@pytest.mark.parametrize("dtype", [0, 1])
def test_row_complete_layernorm_epilogues_msa(dtype, variant, use_ctx):
    """256 MSA channels: the GEMMs that produce the cotangent of a LayerNorm output in the MSA stack and in the outer
    product mean finish the LayerNorm backward on 64 x 256 tiles.  s * r = 171 rows: two full tiles and a ragged one of
    43 rows; the Multimer ordering's outer product mean normalises the block's input instead of the stack's output."""
    dims, table, inp = _case("tiny", dtype=dtype, s=9, r=19, c_m=256, c_z=32, h_msa=8, d_msa=32, h_pair=2, d_pair=16,
                             c_tri=16, c_opm=8, n_trans=2, variant=variant)
    table, n = param_table(dims)
    inp = make_inputs(dims, table, n, ("random_residues", 0.1), 29)
    errs, worst, tol, stats = check_case(dims, table, inp, use_ctx=use_ctx)
    if dtype == 1:
        _assert_small(errs, tol, stats)
    else:
        _assert(errs, worst, tol, stats)


@pytest.mark.parametrize("use_ctx", [True, False])
@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("variant", [1, 2])
def test_block_orderings_small(variant, dtype, use_ctx):
    """The AlphaFold2 (Figure 1(a)) and Multimer (Figure 1(b)) orderings of the same sub-operations,
    ragged shape, fp32 and bf16, with saved activations and with the forward recomputed."""
    dims, table, inp = _case("tiny", dtype=dtype, s=37, r=150, c_m=64, c_z=32, h_msa=2, d_msa=16, h_pair=4,
                             d_pair=8, c_tri=24, c_opm=16, n_trans=2, variant=variant)
    table, n = param_table(dims)
    inp = make_inputs(dims, table, n, ("random_residues", 0.07), 5)
    errs, worst, tol, stats = check_case(dims, table, inp, use_ctx=use_ctx)
    if dtype == 1:
        _assert_small(errs, tol, stats)
    else:
        _assert(errs, worst, tol, stats)


@pytest.mark.parametrize("variant", [1, 2])
def test_block_orderings_af2_initial_bf16(variant):
    """The other two orderings at the benchmark shape, bf16, every output element."""
    dims, table, inp = _case("af2_initial", variant=variant)
    _assert(*check_case(dims, table, inp))


# Gradients against the PLAIN oracle (its own ReLU decisions everywhere): the few decisions that differ inside
# the pre-activation's error band change their elements' gradients by O(1), so this comparison is outside the
# tolerance by construction (tests/test_bf16_relu_band.py shows 1e-1 on a transition's input cotangent from the
# flips alone).  It is bounded all the same, so that the unmatched figure is pinned: measured 4e-2..1.1e-1.
PLAIN_BF16_BOUND = 0.2


def _assert_plain(stats):
    plain = stats["plain"]
    worst = max(plain, key=plain.get)
    print("unmatched ReLU decisions: worst %s = %.3e" % (worst, plain[worst]))
    assert plain[worst] <= PLAIN_BF16_BOUND, (worst, plain[worst])


def test_af2_initial_bf16():
    """Config 2: the benchmark workload at full size, bf16 path, every output element: forward against the
    plain oracle, backward under validated ReLU decisions, and the plain-oracle backward bounded."""
    dims, table, inp = _case("af2_initial")
    errs, worst, tol, stats = check_case(dims, table, inp, plain_backward=True)
    _assert(errs, worst, tol, stats)
    _assert_plain(stats)


def test_af2_initial_bf16_one_stream():
    """Config 2 on one stream, side by side on the handle's own, and one branch after the other: a branch that has the chip to
    itself takes the parameter-gradient GEMM with two wave groups; every output element against the oracle."""
    dims, table, inp = _case("af2_initial")
    _assert(*check_case(dims, table, inp, two_streams=False))
    errs, worst, tol, stats = check_case(dims, table, inp, two_streams=False, timed=True)
    assert any("gemm_dwx_kernel<2>" in v for v in stats["kernels"].values()), stats["kernels"]
    _assert(errs, worst, tol, stats)


def test_ragged_shapes_one_stream_bf16():
    """The ragged shape on one stream (bf16): tails in m, n and k of the two-wave-group parameter-gradient GEMM."""
    dims, table, inp = _case("tiny", dtype=1, s=37, r=150, c_m=64, c_z=32, h_msa=2, d_msa=16, h_pair=4,
                             d_pair=8, c_tri=24, c_opm=16, n_trans=2)
    table, n = param_table(dims)
    inp = make_inputs(dims, table, n, ("random_residues", 0.07), 5)
    errs, worst, tol, stats = check_case(dims, table, inp, two_streams=False, timed=True)
    assert any("gemm_dwx_kernel<2>" in v for v in stats["kernels"].values()), stats["kernels"]
    _assert_small(errs, tol, stats)


@pytest.mark.parametrize("two_streams", [True, False])
def test_random_small_shapes_fp32(two_streams):
    """Six seeded random draws of every size parameter (sequences 3..69, residues 8..200, channel widths, head
    counts and dimensions, hidden sizes, block ordering), fp32 path at 1e-4, with the branches on two streams and
    on one (side by side on the handle's own stream but for the smallest)."""
    rng = np.random.default_rng(123)
    for i in range(6):
        dims, _, _ = dims_for("tiny")
        dims.update(dtype=0, s=int(rng.integers(3, 70)), r=int(rng.choice([8, 24, 40, 72, 136, 200])),
                    c_m=int(rng.choice([32, 64, 128])), c_z=int(rng.choice([16, 32, 64, 128])),
                    h_msa=int(rng.choice([1, 2, 4])), d_msa=int(rng.choice([8, 16, 32])),
                    h_pair=int(rng.choice([1, 2, 4])), d_pair=int(rng.choice([8, 16, 32])),
                    c_tri=int(rng.choice([8, 16, 24, 64])), c_opm=int(rng.choice([8, 16, 32])),
                    n_trans=int(rng.choice([2, 4])), variant=int(rng.choice([0, 0, 1, 2])))
        table, n = param_table(dims)
        inp = make_inputs(dims, table, n, ("random_residues", 0.1), 100 + i)
        errs, worst, tol, _ = check_case(dims, table, inp, two_streams=two_streams)
        assert errs[worst] <= tol, "draw %d %s: worst %s = %.3e" % (i, dims, worst, errs[worst])


def test_af2_initial_fp32():
    dims, table, inp = _case("af2_initial", dtype=0)
    _assert(*check_case(dims, table, inp))


def test_recompute_and_single_stream_match():
    """Backward with ctx == NULL (internal recompute), both branches on one stream, and the
    parameter-gradient kernels on library-owned side streams (PE_OPT_SIDE_STREAMS) give
    bit-identical results to the two-stream, saved-ctx run.  One exception: where one stream's branches run one after the
    other (a timed call), the bf16 parameter-gradient GEMMs split their k range over two wave groups, so their fp32 sums are taken
    in another order there: parameter gradients agree to fp32 rounding instead."""
    import torch
    from tests.gpu_util import BlockRun
    dims, table, inp = _case("tiny", dtype=1, s=24, r=48)
    table, n = param_table(dims)
    inp = make_inputs(dims, table, n, ("last_residues", 5), 9)
    outs = []
    for two, use_ctx, side, timed in ((True, True, False, False), (False, True, False, True), (True, False, False, False),
                                      (True, True, True, False), (True, False, True, False), (False, True, False, False)):
        run = BlockRun(dims, inp, two_streams=two)
        if timed:
            run.h.set_option(3, 1)
        if side:
            run.h.set_option(4, 1)
        run.fwd()
        if not use_ctx:
            run.sync()          # zero_() runs on torch's stream, the forward on the run's own streams
            run.ctx.zero_()
            run.sync()
        run.bwd(use_ctx=use_ctx)
        run.sync()
        outs.append([t.clone() for t in (run.msa_out, run.pair_out, run.d_msa_in, run.d_pair_in, run.d_params)])
    for idx, other in enumerate(outs[1:], 1):
        for a, b in zip(outs[0][:4], other[:4]):
            assert torch.equal(a, b)
        if idx == 1:    # one branch after the other
            scale = outs[0][4].abs().max().item()
            assert (outs[0][4] - other[4]).abs().max().item() <= 1e-5 * scale
        else:
            assert torch.equal(outs[0][4], other[4])


@pytest.mark.slow
@pytest.mark.parametrize("use_ctx", [True, False])
def test_af2_finetune_bf16(use_ctx):
    """Config 4: fine-tuning shape (s=512, r=384), bf16 path, every output element; with the saved
    activations and with ctx == NULL (the backward call recomputes the forward: the block at full recompute)."""
    dims, table, inp = _case("af2_finetune")
    _assert(*check_case(dims, table, inp, use_ctx=use_ctx))


@pytest.mark.parametrize("dtype", [0, 1])
def test_masked_edge_cases(dtype):
    """An all-ones mask, and all residues masked but one (column attention sees no valid key at a masked
    residue; row and triangle attention have a single valid key)."""
    for recipe in (("none", 0), ("last_residues", 15)):
        dims, table, inp = _case("tiny", dtype=dtype)
        table, n = param_table(dims)
        inp = make_inputs(dims, table, n, recipe, 21)
        errs, worst, tol, stats = check_case(dims, table, inp)
        if dtype == 1:
            _assert_small(errs, tol, stats)
        else:
            _assert(errs, worst, tol, stats)


@pytest.mark.parametrize("dtype", [0, 1])
def test_first_key_tile_fully_masked(dtype):
    """The first 70 of 150 residues masked: the first 64-key tile of every row / triangle attention holds no
    valid key (the online softmax starts from an empty tile and meets its first finite logit later), queries
    at masked residues included; column attention has whole columns without a valid key."""
    dims, table, inp = _case("tiny", dtype=dtype, s=37, r=150, c_m=64, c_z=32, h_msa=2, d_msa=16, h_pair=4,
                             d_pair=8, c_tri=24, c_opm=16, n_trans=2)
    table, n = param_table(dims)
    inp = make_inputs(dims, table, n, ("first_residues", 70), 61)
    errs, worst, tol, stats = check_case(dims, table, inp)
    if dtype == 1:
        _assert_small(errs, tol, stats)
    else:
        _assert(errs, worst, tol, stats)


@pytest.mark.parametrize("s,r", [(40, 41), (33, 20)])
def test_fp32_values_beyond_the_largest_bf16_number(s, r):
    """fp32 operands that round to infinity in bf16 (3.4e38; the largest bf16 number is 3.39e38) in the GEMMs of the backward pass that split
    them into bf16 terms: one weight of both transitions, w1[0][0], against a LayerNorm output that is 2e-38 there (gain 0, offset 2e-38) on
    the way forward and a cotangent of order 1e-36 (outgoing weights 1e-36) on the way back.  Everything stays of order one to a thousand."""
    dims, table, inp = _case("af2_initial", dtype=0, s=s, r=r)
    at = {e["name"]: e for e in table}

    def entry(name):
        e = at[name]
        return inp["params"][e["offset"]:e["offset"] + int(np.prod(e["shape"]))].reshape(e["shape"])

    for t in ("mtrans", "ptrans"):
        entry(t + ".ln.g")[0] = 0.0
        entry(t + ".ln.b")[0] = 2e-38
        entry(t + ".w1")[0, 0] = 3.4e38
        entry(t + ".w2")[0, :] = 1e-36
    errs, worst, tol, stats = check_case(dims, table, inp)
    _assert(errs, worst, tol, stats)


def test_fp32_outer_product_cotangents_on_fp32_mfmas():
    """The outer product's cotangents are not split into bf16 terms (LayerNorm gradients below them lose accuracy)."""
    dims, table, inp = _case("extra_msa", dtype=0, s=300, r=64)
    names = _kernels_by_label(BlockRun(dims, inp))
    assert names["opm da"] == {"gemm_kernel<kc,kc,vec,EpiPartialF32>"}, names["opm da"]
    assert names["opm db"] == {"gemm_kernel<kc,xc,vec,EpiPartialF32>"}, names["opm db"]


def _tensor(table, flat, name):
    e = [x for x in table if x["name"] == name][0]
    return flat[e["offset"]:e["offset"] + int(np.prod(e["shape"]))].reshape(e["shape"])


def _param_grads(dims, inp):
    """Flat parameter gradients of the HIP path and of the oracle under the path's (validated) ReLU decisions."""
    args = (dims, inp["params"], inp["msa"], inp["pair"], inp["msa_mask"], inp["pair_mask"])
    _, _, _, inter = ev.block_fwd(*args, want_cache=False)
    run = BlockRun(dims, inp)
    run.fwd(use_ctx=True)
    run.sync()
    on, stats, _ = relu_decisions(dims, run, inter)
    assert all(st["flips_outside"] == 0 for st in stats.values()), stats
    _, _, cache, _ = ev.block_fwd(*args, relu_on=on)
    _, _, ref, _ = ev.block_bwd(dims, cache, inp["d_msa_out"], inp["d_pair_out"])
    run.bwd()
    run.sync()
    return to_np(run.d_params), ref


def test_fp32_cotangents_too_small_for_three_bf16_terms():
    """Cotangents of a hidden unit of about 2e-38 (outgoing weights 1e-39) against a weight of 1e38: three bf16 terms hold 13 bits of them
    (bf16 ends at 2^-133), the products are of order one and make up the gradients of the LayerNorm offset and gain."""
    dims, table, inp = _case("af2_initial", dtype=0, s=40, r=41)
    for t in ("mtrans", "ptrans"):
        _tensor(table, inp["params"], t + ".ln.g")[0] = 0.0
        _tensor(table, inp["params"], t + ".ln.b")[0] = 2e-38
        _tensor(table, inp["params"], t + ".w1")[0, 0] = 1e38
        _tensor(table, inp["params"], t + ".w2")[0, :] = np.float32(1e-39)
    errs, worst, tol, stats = check_case(dims, table, inp)
    _assert(errs, worst, tol, stats)


@pytest.mark.parametrize("value,scale", [(2.0123e-38, 1.0), (3.4e38, 1e-4)])
def test_fp32_activations_without_three_bf16_terms(value, scale):
    """A LayerNorm output channel of 2e-38 (bf16 terms hold 9 bits) or 3.4e38 (infinity in bf16) in every position: that row of the first
    transition weight's gradient, split along an odd number of positions, rows fewer than a tile's, against float64."""
    dims, table, inp = _case("extra_msa", dtype=0, s=41, r=53)
    inp["d_msa_out"] *= scale
    inp["d_pair_out"] *= scale
    value = float(np.float32(value))
    for t in ("mtrans", "ptrans"):
        _tensor(table, inp["params"], t + ".ln.g")[0] = 0.0
        _tensor(table, inp["params"], t + ".ln.b")[0] = value
        if value > 1:
            _tensor(table, inp["params"], t + ".w1")[0, :] *= 1e-38
    names = _kernels_by_label(BlockRun(dims, inp))
    assert names["trans dW1"] == {"gemm_kernel<xc,xc,vec,EpiPartial>"}, names["trans dW1"]
    got, ref = _param_grads(dims, inp)
    for t in ("mtrans", "ptrans"):
        a, b = _tensor(table, got, t + ".w1")[0], _tensor(table, ref, t + ".w1")[0]
        assert np.linalg.norm(a - b) <= TOL[0] * np.linalg.norm(b), (t, np.linalg.norm(a - b) / np.linalg.norm(b))


def test_fp32_weights_beyond_the_largest_bf16_number():
    """Attention output weights and triangle operands of 3.4e38 against values of 1e-38 on their other side: the attention and triangle
    cotangents that go through bf16 terms, in every kernel that has them, with ragged tiles."""
    dims, table, inp = _case("af2_initial", dtype=0, s=46, r=183)
    inp["d_msa_out"] *= 1e-6
    inp["d_pair_out"] *= 1e-6
    for t in ("row", "col", "tas", "tae"):
        _tensor(table, inp["params"], t + ".w_v")[:, 0] *= 1e-38
        w = _tensor(table, inp["params"], t + ".w_o")
        w[0, :] = np.where(w[0, :] < 0, -3.4e38, 3.4e38)
    for t in ("tmo", "tmi"):
        _tensor(table, inp["params"], t + ".w_ap")[:, 0] *= 1e-38
        _tensor(table, inp["params"], t + ".b_ap")[0] = 0.0
        _tensor(table, inp["params"], t + ".w_bp")[:, 0] = 0.0
        _tensor(table, inp["params"], t + ".b_bp")[0] = 3.4e38
        _tensor(table, inp["params"], t + ".w_bg")[:, 0] = 0.0
        _tensor(table, inp["params"], t + ".b_bg")[0] = 200.0
    names = _kernels_by_label(BlockRun(dims, inp))
    assert names["attn dog+pre"] == {"gemm_kernel<kc,kc,vec,EpiAttnPre>", "gemm64_kernel<EpiAttnPre>"}, names["attn dog+pre"]
    assert all(k.endswith("EpiTmGateBwd>") for k in names["trimul da+gate"]), names["trimul da+gate"]
    errs, worst, tol, stats = check_case(dims, table, inp)
    _assert(errs, worst, tol, stats)


def test_fp32_long_contraction_of_one_sign():
    """The second transition weight's gradient over 3072 positions per split of non-negative operands (hidden units, cotangents made
    positive): its error against float64 has no side.  Half a bit to one side per 16 positions would be 96 x 2^-24 = 6e-6 of every element on average;
    a rounding per 16 positions and per split of the sum that adds the 32 splits up is at most 224 x 2^-24 = 1.3e-5."""
    import torch
    dims, table, inp = _case("af2_initial", dtype=0, s=256, r=384)
    inp["d_msa_out"] = np.abs(inp["d_msa_out"])
    inp["d_pair_out"] = np.zeros_like(inp["d_pair_out"])
    run = BlockRun(dims, inp)
    run.fwd(use_ctx=True)
    run.bwd()
    run.sync()
    e = [x for x in pe.ctx_table(dims) if x["name"] == "mtrans.h"][0]
    h = run.ctx[e["offset_bytes"]:e["offset_bytes"] + 4 * e["count"]].view(torch.float32).reshape(256 * 384, -1)
    g = run.d_msa_out.reshape(256 * 384, -1)
    ref = torch.zeros(h.shape[1], g.shape[1], dtype=torch.float64, device="cuda")
    for i in range(0, 256 * 384, 8192):
        ref += h[i:i + 8192].double().t().contiguous() @ g[i:i + 8192].double()
    got = torch.from_numpy(_tensor(table, to_np(run.d_params), "mtrans.w2")).cuda()
    err = (got - ref) / ref.abs().clamp_min(1e-300)
    mean, rms = float(err.mean()), float((err * err).mean().sqrt())
    print("mean %.3e rms %.3e max %.3e" % (mean, rms, float(err.abs().max())))
    assert abs(mean) <= 1e-6 and float(err.abs().max()) <= 1.3e-5, (mean, rms)


@pytest.mark.parametrize("dtype", [0, 1])
def test_large_magnitude_inputs(dtype):
    """Inputs drawn 8 times wider (N(0, 64)): LayerNorm inputs of large magnitude and, through the un-normalised
    residual paths, logits whose running maximum moves by tens between key tiles (the online-softmax rescale);
    s = 70 and r = 150 give two and three key tiles."""
    dims, table, inp = _case("tiny", dtype=dtype, s=70, r=150, c_m=64, c_z=32, h_msa=2, d_msa=16, h_pair=4,
                             d_pair=8, c_tri=24, c_opm=16, n_trans=2)
    table, n = param_table(dims)
    inp = make_inputs(dims, table, n, ("random_residues", 0.07), 62, scale=8.0)
    errs, worst, tol, stats = check_case(dims, table, inp)
    if dtype == 1:
        _assert_small(errs, tol, stats)
    else:
        _assert(errs, worst, tol, stats)


def test_peaked_softmax_fp32():
    """Query / key weights scaled by 3: logits nine times wider (tens in the base-2 domain) with a different
    winner per key tile, so the running maximum of the online softmax jumps by many units from tile to tile and
    the rescale factor of the earlier tiles gets tiny (fp32 path: the comparison is sharp there)."""
    dims, table, inp = _case("tiny", dtype=0, s=70, r=150, c_m=64, c_z=32, h_msa=2, d_msa=16, h_pair=4,
                             d_pair=8, c_tri=24, c_opm=16, n_trans=2)
    table, n = param_table(dims)
    inp = make_inputs(dims, table, n, ("random_residues", 0.07), 63)
    for e in table:
        if e["name"].endswith((".w_q", ".w_k")):
            k = int(np.prod(e["shape"]))
            inp["params"][e["offset"]:e["offset"] + k] *= 3.0
    inp["params"] = inp["params"].astype(np.float32).astype(np.float64)
    errs, worst, tol, stats = check_case(dims, table, inp)
    _assert(errs, worst, tol, stats)


@pytest.mark.parametrize("s,r", [(1, 1), (1, 9), (9, 1), (2, 130)])
def test_degenerate_sizes(s, r):
    """A single sequence, a single residue, both, and a 2-row MSA over more than one tile of
    residues: every contraction and softmax collapses to length 1 somewhere (fp32 path)."""
    dims, table, inp = _case("tiny", dtype=0, s=s, r=r)
    table, n = param_table(dims)
    inp = make_inputs(dims, table, n, ("none", 0), 23)
    _assert(*check_case(dims, table, inp))


def test_bad_arguments_return_errors():
    import torch
    import paper_2211_00235_amd as pe
    from tests.gpu_util import BlockRun
    dims, table, inp = _case("tiny")
    run = BlockRun(dims, inp)
    with pytest.raises(pe.PEError, match="aliases"):
        pe.block_fwd(run.h, dims, run.msa, run.pair, run.msa_mask, run.pair_mask, run.params, run.msa, run.pair_out,
                     run.ctx, run.ws)
    # buffers the call writes may not overlap any other buffer: d_params on params, ctx inside the workspace
    with pytest.raises(pe.PEError, match="aliases"):
        pe.block_bwd(run.h, dims, run.msa, run.pair, run.msa_mask, run.pair_mask, run.params, run.d_msa_out,
                     run.d_pair_out, run.d_msa_in, run.d_pair_in, run.params, run.ctx, run.ws)
    with pytest.raises(pe.PEError, match="aliases"):
        pe.block_fwd(run.h, dims, run.msa, run.pair, run.msa_mask, run.pair_mask, run.params, run.msa_out,
                     run.pair_out, run.ws, run.ws)
    with pytest.raises(pe.PEError, match="aliases"):
        pe.block_bwd(run.h, dims, run.msa, run.pair, run.msa_mask, run.pair_mask, run.params, run.d_msa_out,
                     run.d_pair_out, run.d_msa_in, run.d_pair_in, run.d_params, run.ctx, run.ctx)
    small = torch.empty(4096, dtype=torch.uint8, device="cuda")
    with pytest.raises(pe.PEError, match="workspace too small"):
        pe.block_fwd(run.h, dims, run.msa, run.pair, run.msa_mask, run.pair_mask, run.params, run.msa_out,
                     run.pair_out, run.ctx, small)
    bad = dict(dims, c_m=30)
    with pytest.raises(pe.PEError, match="unsupported dims.*multiples of 8"):
        pe.block_fwd(run.h, bad, run.msa, run.pair, run.msa_mask, run.pair_mask, run.params, run.msa_out,
                     run.pair_out, run.ctx, run.ws)


@pytest.mark.parametrize("dtype", [0, 1])
def test_global_column_attention_small(dtype):
    """Extra-MSA block variant (global column attention) at a small ragged shape."""
    dims, table, inp = _case("tiny", dtype=dtype, s=70, r=45, c_m=32, h_msa=4, d_msa=8, col_global=1)
    table, n = param_table(dims)
    inp = make_inputs(dims, table, n, ("random_rows", 0.1), 31)
    errs, worst, tol, stats = check_case(dims, table, inp)
    if dtype == 1:
        _assert_small(errs, tol, stats)
    else:
        _assert(errs, worst, tol, stats)


@pytest.mark.parametrize("h_msa,s,r,dtype", [(3, 700, 20, 0), (8, 300, 24, 0), (1, 1100, 12, 0), (5, 333, 16, 1)])
def test_global_column_attention_head_counts_and_sequence_chunks(h_msa, s, r, dtype):
    """Global column attention with head counts that do not divide a workgroup's threads (idle sequence lanes in the
    reductions over s) and sequence lengths of several chunks with a ragged last one."""
    dims, table, inp = _case("tiny", dtype=dtype, s=s, r=r, c_m=32, h_msa=h_msa, d_msa=8, col_global=1)
    table, n = param_table(dims)
    inp = make_inputs(dims, table, n, ("random_rows", 0.1), 37 + h_msa)
    errs, worst, tol, stats = check_case(dims, table, inp)
    if dtype == 1:
        _assert_small(errs, tol, stats)
    else:
        _assert(errs, worst, tol, stats)


def _kernel_launches(run, use_ctx=True):
    """One forward and backward pass with per-kernel timing on: launches by kernel name."""
    run.h.set_option(3, 1)      # PE_OPT_KERNEL_TIMING
    run.fwd(use_ctx=use_ctx)
    run.bwd(use_ctx=use_ctx)
    run.sync()
    out = {}
    for e in run.h.timing_collect():
        out[e["kernel"]] = out.get(e["kernel"], 0) + e["launches"]
    run.h.set_option(3, 0)
    return out


def _check_walking_backward(dims, inp, table, launches):
    """Gradients only, against the oracle under the path's own ReLU decisions and at the tolerance of the bf16 path; the
    forward pass and the validity of the decisions are not these tests' (the band of tests/parity.py is calibrated on
    fewer units than a pair transition has here: r^2 x 64 of them put the largest pre-activation error of the 16-channel
    forward pass at 5e-2 rms).  launches: how many attentions of the block take the walking kernel."""
    run = BlockRun(dims, inp)
    assert _kernel_launches(run).get("attn_bwd_walk_kernel", 0) == launches
    run.d_params.zero_()
    run.sync()
    run.fwd(use_ctx=True)
    run.bwd(use_ctx=True)
    run.sync()
    args = (dims, inp["params"], inp["msa"], inp["pair"], inp["msa_mask"], inp["pair_mask"])
    inter = ev.block_fwd(*args, want_cache=False)[3]
    _, _, cache, _ = ev.block_fwd(*args, relu_on=relu_decisions(dims, run, inter)[0])
    dm, dz, g, _ = ev.block_bwd(dims, cache, inp["d_msa_out"], inp["d_pair_out"])
    errs = {"d_msa_in": rel_err(to_np(run.d_msa_in), dm), "d_pair_in": rel_err(to_np(run.d_pair_in), dz)}
    errs.update({"d_params." + k: v for k, v in param_errors(to_np(run.d_params), g, table).items()})
    worst, val = worst_scaled(errs, {"d_params." + e["name"]: int(np.prod(e["shape"])) for e in table})
    assert val <= TOL[1], (worst, errs[worst])


@pytest.mark.parametrize("h_msa,s,r,mask", [(4, 1050, 33, "random_rows"), (8, 600, 128, "random_residues"),
                                            (8, 271, 130, "random_rows"), (8, 200, 290, "random_residues"),
                                            (8, 192, 384, "random_rows"), (8, 545, 17, "random_rows")])
def test_row_attention_backward_over_many_rows(h_msa, s, r, mask):
    """Head dimension 8 and enough rows for the backward kernel that walks through them (attn_walk_splits > 0): one key
    block and several, one query tile (two of the three wave groups own none), ragged last key block / key tile / query
    tile, splits of unequal length, rows whose keys are all masked and rows with some of them masked."""
    dims, table, inp = _case("tiny", dtype=1, s=s, r=r, c_m=32, h_msa=h_msa, d_msa=8, col_global=1)
    table, n = param_table(dims)
    inp = make_inputs(dims, table, n, (mask, 0.1), 41 + h_msa)
    _check_walking_backward(dims, inp, table, 1)


def test_triangle_attention_backward_over_many_rows():
    """Pair heads of dimension 8 send both triangle attentions through the walking kernel: positions and key mask strided
    the other way round at the ending node, a ragged third key block, bias gradient in the LayerNorm epilogue's order."""
    dims, table, inp = _case("tiny", dtype=1, s=4, r=257, c_m=32, c_z=32, h_pair=8, d_pair=8)
    table, n = param_table(dims)
    inp = make_inputs(dims, table, n, ("random_residues", 0.1), 43)
    _check_walking_backward(dims, inp, table, 2)


def test_attention_logits_far_below_zero():
    """Every logit of the row attention near -300 (a pair bias that is the same for all keys, to which the softmax is
    indifferent): the first reference maximum is that low, and 2^(0 - reference) is not a finite factor."""
    dims, table, inp = _case("tiny", dtype=0, s=6, r=70)
    table, n = param_table(dims)
    inp = make_inputs(dims, table, n, ("random_residues", 0.1), 51)
    for name, value in (("row.ln_z.g", 0.0), ("row.ln_z.b", 1.0), ("row.w_bias", -300.0)):
        e = next(e for e in table if e["name"] == name)
        w = inp["params"][e["offset"]:e["offset"] + int(np.prod(e["shape"]))].reshape(e["shape"])
        w[0] = value     # channel 0
    run = BlockRun(dims, inp)
    run.fwd()
    run.sync()
    m, z, _, _ = ev.block_fwd(dims, inp["params"], inp["msa"], inp["pair"], inp["msa_mask"], inp["pair_mask"], want_cache=False)
    assert rel_err(to_np(run.msa_out), m) < TOL[0] and rel_err(to_np(run.pair_out), z) < TOL[0]


def _entry(inp, table, name):
    """View of one parameter in inp["params"]."""
    e = next(e for e in table if e["name"] == name)
    return inp["params"][e["offset"]:e["offset"] + int(np.prod(e["shape"]))].reshape(e["shape"])


@pytest.mark.parametrize("h_msa,d_msa,s,r,dtype", [(2, 32, 37, 150, 1), (4, 16, 21, 65, 1), (2, 32, 13, 70, 0)])
def test_attention_without_a_bias_is_one_with_a_zero_bias(h_msa, d_msa, s, r, dtype):
    """The column attention of a transposed MSA against the row attention with a bias of zero: forward and backward go through
    the kernels without and with a bias, which do the same arithmetic, so outputs and cotangents are the same bits (adding an
    exact zero to a logit changes nothing).  The other sub-operations pass the MSA through: their output weights are zero."""
    over = dict(c_m=64, h_msa=h_msa, d_msa=d_msa)
    dims, table, inp = _case("tiny", dtype=dtype, s=s, r=r, **over)
    table, n = param_table(dims)
    inp = make_inputs(dims, table, n, ("random_residues", 0.1), 67)
    for name in ("row.w_bias", "row.b_o", "col.b_o", "mtrans.w2", "mtrans.b2", "opm.w_o"):
        _entry(inp, table, name)[...] = 0.0
    tdims, ttable, tinp = _case("tiny", dtype=dtype, s=r, r=s, **over)
    tinp["params"] = inp["params"].copy()
    for k in ("msa", "d_msa_out"):
        tinp[k] = np.ascontiguousarray(inp[k].transpose(1, 0, 2))
    tinp["msa_mask"] = np.ascontiguousarray(inp["msa_mask"].T)
    for a, b in (("row.ln_m.g", "col.ln.g"), ("row.ln_m.b", "col.ln.b")) + tuple(("row." + w, "col." + w) for w in ("w_q", "w_k", "w_v", "w_g", "b_g", "w_o")):
        _entry(tinp, ttable, b)[...] = _entry(inp, table, a)
    _entry(inp, table, "col.w_o")[...] = 0.0
    _entry(tinp, ttable, "row.w_o")[...] = 0.0
    row, col = BlockRun(dims, inp), BlockRun(tdims, tinp)
    for run in (row, col):
        run.fwd()
        run.bwd()
        run.sync()
    for k in ("msa_out", "d_msa_in"):
        a, b = to_np(getattr(row, k)), to_np(getattr(col, k)).transpose(1, 0, 2)
        assert np.array_equal(a, b), (k, rel_err(a, b))
    base = inp["msa"] if dtype == 1 else inp["msa"].astype(np.float32)
    assert rel_err(to_np(row.msa_out), base) > 1e-2      # the attention does take part


@pytest.mark.parametrize("dtype,sign", [(1, -1.0), (1, 1.0), (0, -1.0)])
def test_attention_with_a_large_log_sum_exp(dtype, sign):
    """Every logit of the row and the column attention near -300 or 300, forward and backward: channel 0 of q and k is a
    constant, exact in bf16, that adds the same to every logit (the softmax is indifferent to it, lse is not), the other
    channels are as usual.  The constant comes from a normalised channel without gain, so the cotangent that reaches the MSA
    does not see it; the parameters behind that channel are not compared (their exact gradients are sums that cancel)."""
    dims, table, inp = _case("tiny", dtype=dtype, s=39, r=70, c_m=64, h_msa=2, d_msa=32)
    table, n = param_table(dims)
    inp = make_inputs(dims, table, n, ("random_residues", 0.1), 73)
    for at, ln in (("row", "row.ln_m"), ("col", "col.ln")):
        _entry(inp, table, ln + ".g")[0], _entry(inp, table, ln + ".b")[0] = 0.0, 1.0
        for w, v in (("w_q", sign * 42.5), ("w_k", 40.0)):
            m = _entry(inp, table, "%s.%s" % (at, w))      # [channel][head * 32 + position]
            m[:, ::32] = 0.0
            m[0, :] = 0.0
            m[0, ::32] = v
    for name in ("mtrans.w2", "mtrans.b2"):                # no ReLU decision reaches the cotangent
        _entry(inp, table, name)[...] = 0.0
    run = BlockRun(dims, inp)
    run.fwd()
    run.bwd()
    run.sync()
    for name in ("row.lse", "col.lse"):
        lse = run.ctx_entry(name)
        assert np.all((sign * lse > 250.0) | (lse == 0.0)) and np.mean(lse == 0.0) <= 0.1      # 0: no valid key (a masked residue's column)
    args = (dims, inp["params"], inp["msa"], inp["pair"], inp["msa_mask"], inp["pair_mask"])
    m, z, cache, _ = ev.block_fwd(*args)
    dm, dz, _, _ = ev.block_bwd(dims, cache, inp["d_msa_out"], inp["d_pair_out"])
    for got, ref in ((run.msa_out, m), (run.d_msa_in, dm)):
        assert rel_err(to_np(got), ref) < TOL[dtype]


@pytest.mark.parametrize("h_msa,d_msa,s,r,dtype", [(4, 32, 257, 33, 1), (2, 24, 65, 65, 1), (4, 16, 97, 31, 1), (4, 8, 31, 34, 1), (4, 32, 290, 7, 0)])
def test_attention_tiles_and_head_dimensions(h_msa, d_msa, s, r, dtype):
    """Head dimensions of one and two contraction steps, one key more than a staged chunk, a ragged last tile, an odd last batch row."""
    dims, table, inp = _case("tiny", dtype=dtype, s=s, r=r, c_m=64, h_msa=h_msa, d_msa=d_msa)
    table, n = param_table(dims)
    inp = make_inputs(dims, table, n, ("random_residues", 0.1), 53 + d_msa)
    errs, worst, tol, stats = check_case(dims, table, inp)
    _assert(errs, worst, tol, stats)


@pytest.mark.parametrize("name,dtype,over", [("tiny", 0, {}), ("tiny", 1, dict(s=9, r=21, c_tri=24)), ("af2_initial", 1, dict(s=17, r=45)),
                                             ("af2_initial", 1, dict(s=17, r=45, variant=1)), ("af2_initial", 0, dict(s=9, r=34, variant=2)),
                                             ("extra_msa", 1, dict(s=70, r=40))])
def test_forward_without_activations_is_the_same_forward(name, dtype, over):
    """Without a ctx the forward pass leaves out what only a backward pass reads; its outputs are the same bits, also when the
    workspace held NaN before, and a recomputing backward pass after it is the same as one on saved activations."""
    import torch
    dims, table, inp = _case(name, dtype=dtype, **over)
    run = BlockRun(dims, inp)
    run.fwd(use_ctx=True)
    run.bwd(use_ctx=True)
    run.sync()
    outs = ("msa_out", "pair_out", "d_msa_in", "d_pair_in", "d_params")
    ref = {k: getattr(run, k).clone() for k in outs}
    for k in outs[:4]:
        getattr(run, k).fill_(float("nan"))
    run.d_params.zero_()
    run.ws.fill_(0xff)
    run.sync()
    run.fwd(use_ctx=False)
    run.bwd(use_ctx=False)
    run.sync()
    for k in outs:
        assert torch.equal(getattr(run, k), ref[k]), k


@pytest.mark.parametrize("name,dtype,over", [("tiny", 0, {}), ("tiny", 1, {}), ("af2_initial", 1, dict(s=17, r=45)), ("extra_msa", 1, dict(s=70, r=40))])
def test_forward_without_activations_into_unaligned_outputs(name, dtype, over):
    """Outputs that are not 16-byte aligned: without a ctx the MSA stack works in msa_out where it is aligned, and copies
    its result there where it is not.  The same bits, and nothing beside them."""
    import torch
    import paper_2211_00235_amd as pe
    dims, table, inp = _case(name, dtype=dtype, **over)
    run = BlockRun(dims, inp)
    run.fwd(use_ctx=False)
    run.sync()
    n = run.msa_out.numel()
    for shift in (1, 16 // run.msa_out.element_size() // 2):
        buf = torch.full((n + 64,), 7.0, dtype=run.msa_out.dtype, device="cuda")
        out = buf[16 + shift:16 + shift + n]
        assert out.data_ptr() % 16
        run.pair_out.zero_()
        torch.cuda.synchronize()
        pair = run.pair_out.clone()
        pe.block_fwd(run.h, run.dims, run.msa, run.pair, run.msa_mask, run.pair_mask, run.params, out, pair, None, run.ws, run.sm, run.sp)
        run.sync()
        assert torch.equal(out, run.msa_out.reshape(-1))
        assert bool((buf[:16 + shift] == 7.0).all()) and bool((buf[16 + shift + n:] == 7.0).all())


@pytest.mark.parametrize("name,s,r,two_streams,ks", [("af2_initial", 81, 131, False, (256, 128)), ("af2_initial", 9, 33, False, (128,)),
                                                     ("extra_msa", 150, 47, True, (64,))])
def test_row_streaming_gemms(name, s, r, two_streams, ks):
    """The GEMMs whose waves walk through 32-row blocks (pe_rows.h) at each contraction length: a ragged last block, fewer
    blocks than wave slots (more: the two tests below), head-major output of 8 and 32 channels, strided rows (column
    attention, ending node), ReLU decisions on the way out and in."""
    dims, table, inp = _case(name, s=s, r=r)
    table, n = param_table(dims)
    inp = make_inputs(dims, table, n, ("random_residues", 0.1), s + r)
    errs, worst, tol, stats = check_case(dims, table, inp, two_streams=two_streams, timed=True)
    kernels = set().union(*stats["kernels"].values())
    seen = {k.split("K=")[1].rstrip(">") for k in kernels if k.startswith("gemm_rows_kernel")}
    assert {str(k) for k in ks} <= seen, seen
    _assert(errs, worst, tol, stats)


@pytest.mark.parametrize("s,r", [(1, 33), (15, 32), (17, 31), (33, 65), (257, 33), (300, 8)])
def test_outer_product_normaliser(s, r):
    """Counts of sequences per residue pair on 32 x 32 tiles, up to eight waves of 16 sequences: remainders in residues, in a wave's
    sequences and in the waves' rounds; masks that leave some pairs few sequences."""
    dims, table, inp = _case("tiny", dtype=0, s=s, r=r)
    rng = np.random.default_rng(s * 1000 + r)
    inp["msa_mask"] = (rng.random((s, r)) < 0.6).astype(inp["msa_mask"].dtype)
    inp["msa_mask"][0, :] = 1.0
    _, z0, _, _ = ev.block_fwd(dims, inp["params"], inp["msa"], inp["pair"], inp["msa_mask"], inp["pair_mask"], want_cache=False)
    run = BlockRun(dims, inp)
    run.fwd(use_ctx=True)
    run.sync()
    assert rel_err(to_np(run.pair_out), z0) <= TOL[0]


@pytest.mark.parametrize("name,s,r,two_streams,labels", [
    ("af2_initial", 131, 67, False, ("attn out", "trans 2", "attn dog+pre", "opm project")),     # ragged rows, head-major and [(i,p)][(j,q)] operands
    ("af2_initial", 131, 33, True, ("attn out", "attn dog+pre")),                                # strided rows (column attention)
    ("af2_initial", 60, 50, False, ("attn qkvg", "trans 1", "trans dh")),                        # head-major output, ReLU decisions out and in
    ("extra_msa", 260, 33, False, ("trans 1",)),                                                 # one k-step (K = 64)
    ("af2_initial", 5, 128, False, ("trimul out", "trimul da+gate")),                            # a batch of 128 x 128 contractions
])
def test_few_tile_gemms(name, s, r, two_streams, labels):
    """GEMMs of few 64 x 64 tiles with operands by DMA (pe_pipe.h): remainders in rows, one k-step and more, two-level index maps of both
    kinds, a batch, each epilogue that has a kernel there; against the oracle at the path's tolerance."""
    dims, table, inp = _case(name, s=s, r=r)
    table, n = param_table(dims)
    inp = make_inputs(dims, table, n, ("random_residues", 0.1), s + r)
    errs, worst, tol, stats = check_case(dims, table, inp, two_streams=two_streams, timed=True)
    for k in labels:
        assert any(v.startswith("gemm_pipe_kernel") for v in stats["kernels"][k]), (k, stats["kernels"][k])
    _assert(errs, worst, tol, stats)


@pytest.mark.parametrize("s,r,msa,pair", [(5, 127, 32, 32), (5, 128, 32, 32), (5, 129, 32, 64), (129, 127, 32, 32), (129, 131, 64, 64)])
def test_row_complete_epilogues_on_32_and_64_rows(s, r, msa, pair):
    """The row-complete kernels by DMA, which a branch that runs alone takes on every size, at the line between 32-row tiles (up to 16384
    rows) and 64-row tiles, and with remainders in both: LayerNorm forward (pair stack), LayerNorm backward on 128 and 256 channels, with the
    bias path and with the last sum of the pair gradient."""
    dims, table, inp = _case("af2_initial", s=s, r=r)
    errs, worst, tol, stats = check_case(dims, table, inp, two_streams=False, timed=True)
    seen = {k for v in stats["kernels"].values() for k in v if k.startswith("gemm64r") or k.startswith("gemm64w")}
    assert {k.rsplit("DMA=", 1)[-1] for k in seen if k.startswith("gemm64w")} == {"%d>" % msa}, seen
    assert {k.rsplit("DMA=", 1)[-1] for k in seen if k.startswith("gemm64r")} == {"%d>" % pair}, seen
    assert {k.split(",")[1] for k in seen if k.startswith("gemm64r")} == {"MODE=1", "MODE=2"}, seen
    _assert(errs, worst, tol, stats)


def _rows_wave_slots(K, N):
    """Row blocks of 32 that the row-streaming kernel's waves take at once, per panel (launch_rows_np): 256 or 512 workgroups
    of eight waves, shared among the panels in groups of eight workgroups."""
    panel = 128 if K == 128 else 256
    return max(1, 256 * (1 if K == 256 else 2) // (N // panel) // 8) * 8 * 8


def test_row_streaming_gemms_beyond_the_wave_slots():
    """K = 256 and 128 with more row blocks than waves: a wave takes a second block, on the same piece of LDS, and a last one
    that is ragged.  Two streams keep these GEMMs on the tiled kernels, which sum in the same order: outputs and cotangents are
    the same bits."""
    import torch
    s, r = 161, 199
    assert s * r > 32 * _rows_wave_slots(256, 1024) and r * r > 32 * _rows_wave_slots(128, 512)
    dims, table, inp = _case("af2_initial", s=s, r=r)
    one, two = BlockRun(dims, inp, two_streams=False), BlockRun(dims, inp, two_streams=True)
    seen = {k for k in _kernel_launches(one) if k.startswith("gemm_rows_kernel")}
    for form in ("F=3073,K=256", "F=5,K=256", "F=8,K=256", "F=3073,K=128", "F=5,K=128", "F=8,K=128", "F=3136,K=128"):
        assert "gemm_rows_kernel<%s>" % form in seen, (form, seen)
    assert not any(k.startswith("gemm_rows_kernel") for k in _kernel_launches(two))
    for k in ("msa_out", "pair_out", "d_msa_in", "d_pair_in"):
        assert torch.equal(getattr(one, k), getattr(two, k)), k


def test_row_streaming_gemms_beyond_the_wave_slots_at_64_channels():
    """K = 64 with more row blocks than waves.  The transition alone (the other MSA sub-operations have no output), of whose rows
    none knows another: an MSA of 1040 sequences against its two halves, whose rows every wave has one block of at most;
    outputs and cotangents are the same bits.  The head-major projection of the row attention against PyTorch in fp32: bf16
    results, so half a unit in the last place (2^-8 of the value) and the rounding of 64 fp32 products."""
    import torch
    s, r = 1040, 127
    slots = 32 * _rows_wave_slots(64, 256)
    assert s * r > slots >= s * r // 2
    dims, table, inp = _case("extra_msa", s=s, r=r)
    table, n = param_table(dims)
    inp = make_inputs(dims, table, n, ("random_rows", 0.05), 71)
    for name in ("row.w_o", "col.w_o", "opm.w_o"):
        _entry(inp, table, name)[...] = 0.0
    full = BlockRun(dims, inp)
    names = _kernel_launches(full)
    for form in ("F=3073,K=64", "F=5,K=64", "F=8,K=64"):
        assert names.get("gemm_rows_kernel<%s>" % form, 0) > 0, (form, names)
    for h in range(2):
        sl = slice(h * s // 2, (h + 1) * s // 2)
        half_inp = dict(inp, **{k: np.ascontiguousarray(inp[k][sl]) for k in ("msa", "msa_mask", "d_msa_out")})
        half = BlockRun(dict(dims, s=s // 2), half_inp)
        half.fwd()
        half.bwd()
        half.sync()
        for k in ("msa_out", "d_msa_in"):
            assert torch.equal(getattr(full, k)[sl], getattr(half, k)), (k, h)
    H, d, c = dims["h_msa"], dims["d_msa"], dims["c_m"]
    xhat = torch.from_numpy(full.ctx_entry("row.xhat").reshape(s * r, c)).float().cuda()
    qkvg = torch.from_numpy(full.ctx_entry("row.qkvg").reshape(4, H, s * r, d)).float()
    for k, name in enumerate(("row.w_q", "row.w_k", "row.w_v", "row.w_g")):
        w = torch.from_numpy(_entry(inp, table, name)).float().cuda()
        if k == 0:
            w = w * (1.4426950408889634 / d ** 0.5)
        ref = xhat @ w.to(torch.bfloat16).float()
        if k == 3:
            ref = ref + torch.from_numpy(_entry(inp, table, "row.b_g")).float().cuda()
        ref = ref.reshape(s * r, H, d).permute(1, 0, 2).cpu()
        excess = (qkvg[k] - ref).abs() - ref.abs() / 256
        # the scaled query weight is rounded from an fp32 product that may differ in its last place: one bf16 unit of it, rarely
        assert float(excess.max()) < (2e-2 if k == 0 else 1e-4), (name, float(excess.max()))


def test_outer_product_over_many_rows():
    """The outer product's contractions on 256 x 256 tiles (pe_deep.h) in their three operand layouts: 3680 = 14 x 256 + 96
    columns (and a contraction that ends in half a step of 64), a contraction over 3501 rows (an odd tail of 45), ragged last
    tiles in both directions, a last band of fewer than four m-tiles."""
    dims, table, inp = _case("tiny", dtype=1, s=3501, r=115, c_m=32, c_z=32, c_opm=32, h_msa=2, d_msa=8, col_global=1)
    table, n = param_table(dims)
    inp = make_inputs(dims, table, n, ("random_rows", 0.1), 61)
    names = _kernel_launches(BlockRun(dims, inp))
    for form in ("xc,xc", "kc,kc", "kc,xc"):
        assert names.get("gemm_deep_kernel<%s>" % form, 0) == 1, (form, names)
    errs, worst, tol, stats = check_case(dims, table, inp)
    _assert(errs, worst, tol, stats)


def _kernels_by_label(run, branches=3, backward=True):
    """Label -> the kernels that its launches take, of a forward (and backward) pass of the given branches."""
    run.h.set_option(1, branches)      # PE_OPT_BRANCHES
    run.h.set_option(3, 1)             # PE_OPT_KERNEL_TIMING
    run.fwd(use_ctx=backward)
    if backward:
        run.bwd()
    run.sync()
    out = {}
    for e in run.h.timing_collect():
        out.setdefault(e["name"], set()).add(e["kernel"])
    return out


def test_narrow_outputs_keep_their_tiles():
    """A transition over 64 channels: the cotangent of its input has 64 columns and a contraction over 256, which 256 x 256 tiles would
    fill to a quarter (36096 rows are 141 of them, as many as their rule asks for); it stays on the 64-row tiles, while
    the outer product of the same block (3072 x 3072) is on the large ones."""
    dims, table, inp = _case("extra_msa", s=376, r=96)
    names = _kernels_by_label(BlockRun(dims, inp, two_streams=False), branches=1)
    assert names["trans dxhat"] == {"gemm64_kernel<EpiGeneric,F=0>"}, names["trans dxhat"]
    assert names["opm outer"] == {"gemm_deep_kernel<xc,xc>"}, names["opm outer"]


@pytest.mark.parametrize("name,s,r,branch,taken", [
    ("extra_msa", 768, 64, 1, {"attn qkvg": 1, "trans 1": 0, "trans dh": 1}),      # K = 64, N = 256: 768 tiles of 128 x 128
    ("extra_msa", 769, 64, 1, {"attn qkvg": 1, "trans 1": 1, "trans dh": 1}),      # 770
    ("af2_initial", 159, 64, 1, {"attn qkvg": 0, "trans 1": 0, "trans dh": 0}),    # K = 256, N = 1024: 1272 waves
    ("af2_initial", 192, 64, 1, {"attn qkvg": 1, "trans 1": 0, "trans dh": 1}),    # 768 tiles
    ("af2_initial", 193, 64, 1, {"attn qkvg": 1, "trans 1": 1, "trans dh": 1}),    # 776
    ("af2_initial", 256, 64, 1, {"attn qkvg": 1, "trans 1": 1, "trans dh": 1}),    # 2048 waves
    ("af2_initial", 257, 64, 1, {"attn qkvg": 1, "trans 1": 0, "trans dh": 1}),    # 2056
    ("af2_initial", 320, 64, 1, {"attn qkvg": 1, "trans 1": 0, "trans dh": 1}),    # 2560
    ("af2_initial", 321, 64, 1, {"attn qkvg": 1, "trans 1": 1, "trans dh": 1}),    # 2568
    ("af2_initial", 8, 181, 2, {"trimul gate": 1, "trimul dxhat_o": 1}),           # K = 128, N = 128: 32761 rows
    ("af2_initial", 8, 182, 2, {"trimul gate": 0, "trimul dxhat_o": 1}),           # 33124, gemm64_kernel
    ("af2_initial", 8, 221, 2, {"trimul gate": 0, "trimul dxhat_o": 1}),           # 48841: 764 of its workgroups
    ("af2_initial", 8, 222, 2, {"trimul gate": 1, "trimul dxhat_o": 1}),           # 771
])
def test_row_streaming_gemms_where_they_pay(name, s, r, branch, taken):
    """Which GEMMs of one branch go to the row-streaming kernel on either side of each line of its rule (rows_pays), alone on the chip."""
    dims, table, inp = _case(name, s=s, r=r)
    names = _kernels_by_label(BlockRun(dims, inp, two_streams=False), branches=branch)
    got = {k: int(all(n.startswith("gemm_rows_kernel") for n in names[k])) for k in taken}
    assert got == taken, {k: names[k] for k in taken}


@pytest.mark.slow
def test_extra_msa_bf16():
    """Config 3: extra-MSA-stack block (s=1024, r=256, c_m=64, global column attention), bf16."""
    dims, table, inp = _case("extra_msa")
    _assert(*check_case(dims, table, inp))


@pytest.mark.slow
@pytest.mark.parametrize("use_ctx", [True, False])
def test_extra_msa_finetune_depth_against_oracle(use_ctx):
    """Extra-MSA block at the fine-tuning depth of Table 1 (N_extra_seq = 5120) against the float64 oracle,
    element by element, at a residue count the oracle can hold (r = 64): every reduction over the sequence
    axis (outer product mean over 5120 rows, the mean query, keys and values of global column attention, the
    d = 8 row attention at a batch of 5120) runs at its full length; 5 % of the rows masked."""
    dims, mask, _ = dims_for("extra_msa_finetune")
    dims.update(r=64)
    table, n = param_table(dims)
    inp = make_inputs(dims, table, n, mask, 64)
    _assert(*check_case(dims, table, inp, use_ctx=use_ctx))


@pytest.mark.slow
def test_extra_msa_finetune_depth_by_replication():
    """Extra-MSA block at the fine-tuning depth (Table 1: N_extra_seq = 5120, N_res = 384), too
    large for the float64 oracle, checked through a property that holds at any size: an MSA made of
    4 copies of a 1280-row MSA gives the same pair update, the same rows (per copy) and, with the
    MSA cotangent divided by 4 (exact in bf16), the same gradients as the 1280-row problem.  Row
    attention is per row; the mask-weighted mean query, the softmax over 4x duplicated keys and the
    outer product mean (numerator and normaliser both x4, up to its 1e-3 epsilon) are unchanged."""
    import torch
    import paper_2211_00235_amd as pe
    from tests.gpu_util import BlockRun, to_np, rel_err, param_errors
    rep = 4
    base, _, _ = dims_for("extra_msa")
    base.update(s=1280, r=384)
    big = dict(base, s=rep * base["s"])
    table = pe.param_table(base)
    inp = make_inputs(base, table, pe.param_count(base), ("random_rows", 0.05), 7)
    big_inp = dict(inp)
    big_inp["msa"] = np.tile(inp["msa"], (rep, 1, 1))
    big_inp["msa_mask"] = np.tile(inp["msa_mask"], (rep, 1))
    big_inp["d_msa_out"] = np.tile(inp["d_msa_out"], (rep, 1, 1)) / rep

    def run(dims, x):
        r = BlockRun(dims, x)
        r.fwd()
        r.bwd()
        r.sync()
        out = {k: to_np(getattr(r, k)) for k in ("msa_out", "pair_out", "d_msa_in", "d_pair_in", "d_params")}
        del r
        torch.cuda.empty_cache()
        return out

    small = run(base, inp)
    large = run(big, big_inp)
    s = base["s"]
    tol = 1e-2
    assert np.isfinite(large["pair_out"]).all() and np.isfinite(large["d_params"]).all()
    assert rel_err(large["pair_out"], small["pair_out"]) < tol
    assert rel_err(large["d_pair_in"], small["d_pair_in"]) < tol
    # d_msa_in: the two runs round the transition's pre-activation differently (different summation
    # orders upstream), so a ReLU decision at |a| ~ 0 can differ at isolated positions and changes
    # that position's gradient by O(1) (both decisions are valid at bf16); everywhere else the
    # tolerance holds.  Isolated = at most 1e-4 of the (row, residue) positions.
    den = np.max(np.abs(small["d_msa_in"]))
    for k in range(rep):
        assert rel_err(large["msa_out"][k * s:(k + 1) * s], small["msa_out"]) < tol, k
        diff = np.abs(large["d_msa_in"][k * s:(k + 1) * s] * rep - small["d_msa_in"]).max(axis=2) / den
        bad = int((diff >= tol).sum())
        assert bad <= 1e-4 * diff.size, (k, bad)
        assert np.array_equal(large["d_msa_in"][k * s:(k + 1) * s], large["d_msa_in"][:s]), k   # copies are identical
    errs = param_errors(large["d_params"], small["d_params"], table)
    worst = max(errs, key=errs.get)
    assert errs[worst] < tol, (worst, errs[worst])


@pytest.mark.parametrize("name,s,r,variant", [("af2_initial", 17, 45, 0), ("extra_msa", 40, 35, 2), ("tiny", 40, 50, 0)])
def test_one_stream_calls_keep_the_order_of_their_stream(name, s, r, variant):
    """A call with one stream runs its branches side by side, the pair branch on the handle's own stream: inputs written on the caller's stream
    right before a call are what both branches read, and outputs copied on it right after are complete, three times without a host
    synchronisation; equal to the two-stream call's.  Then the same calls captured into a graph on that stream, by a handle that has its own
    stream by then and by one that does not: three replays each with eager work in between."""
    import torch
    dims, table, inp = _case(name, dtype=1, s=s, r=r, variant=variant)
    outs = ("msa_out", "pair_out", "d_msa_in", "d_pair_in", "d_params")
    two = BlockRun(dims, inp)
    two.fwd()
    two.bwd()
    two.sync()
    ref = {k: getattr(two, k).clone() for k in outs}
    run, fresh = BlockRun(dims, inp, two_streams=False), BlockRun(dims, inp, two_streams=False)
    src = {k: getattr(run, k).clone() for k in ("msa", "pair", "params")}
    run.sync()
    got = []
    with torch.cuda.stream(run.sm):
        for _ in range(3):
            for k in src:
                getattr(run, k).zero_()
            for k in outs:
                getattr(run, k).zero_()
            for k in src:
                getattr(run, k).copy_(src[k])
            run.fwd()
            run.bwd()
            got.append({k: getattr(run, k).clone() for k in outs})
    run.sync()
    for g in got:
        for k in outs:
            assert torch.equal(g[k], ref[k]), k
    for r_ in (run, fresh):
        r_.sm = r_.sp = torch.cuda.Stream()      # (the default stream cannot be captured)
        graph = torch.cuda.CUDAGraph()
        r_.d_params.zero_()
        r_.sync()
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=r_.sm):
            r_.fwd()
            r_.bwd()
        for rep in range(3):
            for k in outs:
                getattr(r_, k).zero_()
            r_.ctx.zero_()
            two.fwd()
            two.bwd()
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            for k in outs[:4] if r_ is fresh else outs:      # serial branches sum parameter gradients in another order
                assert torch.equal(getattr(r_, k), ref[k]), (rep, k)


OUTS = ("msa_out", "pair_out", "d_msa_in", "d_pair_in", "d_params")


def _two_stream_outputs(dims, inp):
    run = BlockRun(dims, inp)
    run.fwd()
    run.bwd()
    run.sync()
    return {k: getattr(run, k).clone() for k in OUTS}


def _clear(run):
    for k in OUTS:
        getattr(run, k).zero_()


def _one_stream_run(dims, inp):
    import torch
    run = BlockRun(dims, inp, two_streams=False)
    run.sm = run.sp = torch.cuda.Stream()      # (the default stream cannot be captured)
    return run


@pytest.mark.parametrize("first", [True, False])
def test_first_call_of_a_handle_in_a_capture(first):
    """A handle whose first one-stream calls are captured gives the bits of any other: three replays with eager work in between.  Handles made
    and destroyed, and a call refused for its workspace, while the capture is on leave it whole."""
    import torch
    dims, table, inp = _case("af2_initial", dtype=1, s=64, r=96)
    ref = _two_stream_outputs(dims, inp)
    run, other = _one_stream_run(dims, inp), BlockRun(dims, inp)
    if not first:
        run.fwd()
    ws = run.ws
    graph = torch.cuda.CUDAGraph()
    _clear(run)
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=run.sm):
        run.ws = ws[:256]
        with pytest.raises(pe.PEError):
            run.fwd()
        run.ws = ws
        pe.Handle()
        run.fwd()
        run.ws = ws[:256]
        with pytest.raises(pe.PEError):
            run.bwd()
        run.ws = ws
        run.bwd()
    for rep in range(3):
        _clear(run)
        run.ctx.zero_()
        other.fwd()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for k in OUTS:
            assert torch.equal(getattr(run, k), ref[k]), (rep, k)


def test_one_stream_calls_on_another_stream_during_a_capture():
    """A handle with a call in a capture that has not ended takes an eager call on another stream, which stays out of the capture."""
    import torch
    dims, table, inp = _case("af2_initial", dtype=1, s=17, r=45)
    ref = _two_stream_outputs(dims, inp)
    run, eager = _one_stream_run(dims, inp), _one_stream_run(dims, inp)
    graph = torch.cuda.CUDAGraph()
    for r in (run, eager):
        _clear(r)
    torch.cuda.synchronize()
    eager.h = run.h
    with torch.cuda.graph(graph, stream=run.sm):
        run.fwd()
        eager.fwd()
        run.bwd()
        eager.bwd()
    eager.sync()
    for k in OUTS[:4]:      # (branches one after the other sum parameter gradients in another order)
        assert torch.equal(getattr(eager, k), ref[k]), k
    _clear(eager)
    torch.cuda.synchronize()
    eager.fwd()      # the capture has ended: side by side again
    eager.bwd()
    eager.sync()
    for k in OUTS:
        assert torch.equal(getattr(eager, k), ref[k]), k
    for rep in range(3):
        _clear(run)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for k in OUTS:
            assert torch.equal(getattr(run, k), ref[k]), (rep, k)


def test_refused_calls_leave_no_error_behind():
    """A refused call with a stream and the default stream (NULL), which a handle without a stream of its own once took for its own, and one
    with one stream; a valid call follows each."""
    import torch
    dims, table, inp = _case("tiny", dtype=1, s=40, r=50)
    ref = _two_stream_outputs(dims, inp)
    for streams in ("null", "one"):
        run = _one_stream_run(dims, inp)
        if streams == "null":
            run.sp = torch.cuda.default_stream()
        ws, run.ws = run.ws, run.ws[:256]
        with pytest.raises(pe.PEError):
            run.fwd()
        with pytest.raises(pe.PEError):
            run.bwd()
        run.ws = ws
        run.fwd()
        run.bwd()
        run.sync()
        for k in OUTS:
            assert torch.equal(getattr(run, k), ref[k]), (streams, k)


def test_handles_made_and_destroyed_with_work_pending():
    """Threads that make a handle, call it on a stream of their own and destroy it without waiting, over and over: a handle's stream is passed
    on with the work that is still on it."""
    import threading
    import torch
    dims, table, inp = _case("extra_msa", dtype=1, s=40, r=35)
    ref = _two_stream_outputs(dims, inp)
    runs = [_one_stream_run(dims, inp) for _ in range(4)]
    got, failed = [[] for _ in runs], []

    def work(i):
        try:
            run = runs[i]
            with torch.cuda.stream(run.sm):
                for _ in range(6):
                    run.h = pe.Handle()
                    _clear(run)
                    run.fwd()
                    run.bwd()
                    run.h = None
                    got[i].append({k: getattr(run, k).clone() for k in OUTS})
        except Exception as e:      # noqa: BLE001
            failed.append(e)

    torch.cuda.synchronize()
    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(runs))]
    for th in threads:
        th.start()
    for th in threads:
        th.join()
    torch.cuda.synchronize()
    assert not failed, failed
    for g in got:
        assert len(g) == 6
        for o in g:
            for k in OUTS:
                assert torch.equal(o[k], ref[k]), k


def test_one_stream_calls_stay_on_the_callers_compute_units():
    """A stream with a CU mask keeps the whole call: its branches run one after the other (the parameter gradients are those of a timed
    call, which sums them in the order of a call that runs alone)."""
    import ctypes as C
    import torch
    dims, table, inp = _case("af2_initial", dtype=1, s=64, r=96)
    serial = _one_stream_run(dims, inp)
    serial.h.set_option(3, 1)             # PE_OPT_KERNEL_TIMING
    serial.fwd()
    serial.bwd()
    serial.sync()
    beside = _two_stream_outputs(dims, inp)
    assert not torch.equal(serial.d_params, beside["d_params"])
    st, mask = C.c_void_p(), (C.c_uint32 * 8)(*([0xffffffff] * 4 + [0] * 4))
    L = pe.lib()
    assert L.hipExtStreamCreateWithCUMask(C.byref(st), 8, mask) == 0
    run = BlockRun(dims, inp, two_streams=False)
    run.sm = run.sp = torch.cuda.ExternalStream(st.value)
    run.fwd()
    run.bwd()
    run.sync()
    for k in OUTS:
        assert torch.equal(getattr(run, k), getattr(serial, k)), k
    plain = BlockRun(dims, inp, two_streams=False)      # the default stream has no mask
    plain.fwd()
    plain.bwd()
    plain.sync()
    assert torch.equal(plain.d_params, beside["d_params"])
    assert L.hipStreamDestroy(st) == 0


def test_hip_graph_capture_and_replay():
    """The calls only enqueue work on the caller's streams (no allocation, no host synchronisation,
    no memset nodes), so a caller can capture forward + backward into a HIP graph: three replays,
    with eager runs of a different case in between, each reproduce the eager result bit for bit."""
    import torch
    from tests.gpu_util import BlockRun
    dims, table, inp = _case("tiny", dtype=1, s=24, r=40)
    table, n = param_table(dims)
    inp = make_inputs(dims, table, n, ("random_residues", 0.1), 41)
    other = make_inputs(dims, table, n, ("none", 0), 42)
    run, run2 = BlockRun(dims, inp), BlockRun(dims, other)
    outs = ("msa_out", "pair_out", "d_msa_in", "d_pair_in", "d_params")
    run.fwd()
    run.bwd()
    run.sync()
    ref = {k: getattr(run, k).clone() for k in outs}
    graph = torch.cuda.CUDAGraph()
    run.d_params.zero_()
    run.sync()
    with torch.cuda.graph(graph, stream=run.sm):
        run.fwd()
        run.bwd()
    for rep in range(3):
        for k in outs:
            getattr(run, k).zero_()
        run.ctx.zero_()
        run2.fwd()
        run2.bwd()
        run.sync()
        graph.replay()
        run.sync()
        for k in outs:
            assert torch.equal(getattr(run, k), ref[k]), (rep, k)
