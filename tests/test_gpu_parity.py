"""GPU parity: the HIP path, called through the C-ABI, against the CPU oracle on the same seeded
inputs.  Tolerances (max relative error with the group's rms as floor, tests/parity_util.py):
1e-5 fp32, 2e-2 bf16 inputs / fp32 accumulation, 6e-2 fp8 E4M3.  Integer-valued cases must
match bit for bit.  The full-size mixes are compared on every output element, in the launch
configuration bench.py times.
"""
import numpy as np
import pytest
import torch

from oracle import reference as ref
from paper_2511_00603_amd import binding as B
from paper_2511_00603_amd import runtime as R
from paper_2511_00603_amd.mixrun import StagedMix
from workloads import casts, make_mix

import gpu_util as U
import mix_oracle
from parity_util import TOL, assert_close

pytestmark = pytest.mark.gpu


def check_mix(mix, dtype_name, rows=None, h_scales=None, host_bits=None):
    """One pass on the GPU against the oracle.  fp8 SwiGLU mixes without h_scales: the oracle runs first and its
    own hidden activations give the static scales (amax / 448) that both sides then use."""
    want = None
    if dtype_name == "fp8" and h_scales is None and mix.services[0].kind == "swiglu":
        host_bits = host_bits if host_bits is not None else StagedMix.stage_host(mix, "fp8")
        h_scales = []
        want = mix_oracle.expected(mix, host_bits, dtype_name, rows=rows, calibrated=h_scales)
    staged = StagedMix(mix, dtype_name, U.DEV, s_h=h_scales, host_bits=host_bits)
    staged.run()
    torch.cuda.synchronize()
    got = staged.results()
    if want is None:
        want = mix_oracle.expected(mix, staged.host_bits, dtype_name, rows=rows, h_scales=h_scales)
    tol = TOL[dtype_name]
    worst = 0.0
    assert len(got) == len(want)
    for lg, lw in zip(got, want):
        assert len(lg) == len(lw)
        for (g, label, Y), (g2, label2, Yref) in zip(lg, lw):
            assert (g, label) == (g2, label2)
            if rows is not None:
                Y = Y[rows[g]]
            if dtype_name == "fp8" and label == "H":
                # Stored E4M3 codes.  The oracle rounds fp64 sums, the GPU fp32 MFMA sums, so the same value
                # cannot be handed to both roundings: nearly all codes must agree exactly, a value on a
                # rounding boundary may land one code apart, and near zero (where codes are an absolute
                # 2^-9 * s_h apart) the difference is bounded by the accumulation error instead.
                Y = Y * h_scales[g]
                rms = float(np.sqrt(np.mean(Yref * Yref)))
                step = np.maximum(0.13 * np.maximum(np.abs(Yref), h_scales[g] * 2.0 ** -6), 1e-3 * rms)
                bad = np.argwhere(~(np.abs(Y - Yref) <= step))
                assert len(bad) == 0, "H codes too far apart at %d places, e.g. %s" % (
                    len(bad), [(tuple(int(v) for v in ij), float(Y[tuple(ij)]), float(Yref[tuple(ij)])) for ij in bad[:8]])
                assert np.mean(Y != Yref) < 0.02
                continue
            worst = max(worst, assert_close(Y, Yref, tol, "%s svc %d %s" % (mix.name, g, label)))
    return worst


# A launch with batches of more than 64 rows runs them as block tiles (128 rows) where the planner expects those to finish
# earlier, as it does on a whole chip for the small launches below, and as panel tiles (256 rows) otherwise, always on fewer
# than 128 workgroups: what is said of either kind of tile is tested on a grid that has it.
TALL = {"block": (None, 128), "panel": (64, 256)}


def tall_groups(specs, dtype_name, tiles):
    """Groups on a grid that runs the batches of more than 64 rows as `tiles` ("block", "panel"; fp32: None)."""
    if tiles is None:
        return U.Groups(specs, dtype_name)
    n_workgroups, rows = TALL[tiles]
    G = U.Groups(specs, dtype_name, n_workgroups=n_workgroups)
    assert int(G.plan.classes[-1][1]) == rows and any(int(c) == len(G.plan.classes) - 1 for c in G.plan.tiles["cls"])
    return G


# ---- exactness on integer-valued inputs (layout, indexing, tails) -----------------------------

@pytest.mark.parametrize("dtype_name,tiles", [("f32", None), ("bf16", "block"), ("bf16", "panel"), ("fp8", "block"), ("fp8", "panel")])
def test_small_integers_are_bit_exact(dtype_name, tiles):
    """Small integers: every product and sum is exact in fp32, so the output must be the oracle's, bit for bit,
    after the cast.  fp8 runs with power-of-two per-tensor scales (1/8 for X, 1/4 for W), under which the
    codes, their products and the scale product 2^-5 are all exact."""
    rng = np.random.default_rng(11)
    shapes = [(5, 64, 40), (1, 32, 16), (64, 96, 33), (70, 160, 300), (300, 128, 260), (257, 256, 513), (16, 48, 10)]
    specs = []
    for M, K, N in shapes:
        X = rng.integers(-4, 5, (M, K)).astype(np.float32)
        W = rng.integers(-3, 4, (K, N)).astype(np.float32)
        b = rng.integers(-8, 9, N).astype(np.float32)
        specs.append({"X": X, "W": W, "b": b, "act": "relu", "s_x": 0.125, "s_w": 0.25})
    G = tall_groups(specs, dtype_name, tiles)
    got, want = G.run(), G.expected()
    for (M, K, N), y, yref in zip(shapes, got, want):
        if dtype_name != "f32":
            yref = ref.bf16_decode(ref.bf16_encode(yref))
        assert np.array_equal(y, yref), (dtype_name, M, K, N, np.argwhere(y != yref)[:5])


@pytest.mark.parametrize("dtype_name", ["bf16", "fp8"])
def test_streaming_tiles_in_a_row_add_their_own_bias(dtype_name):
    """Small grid, so that a workgroup streams several tiles of a class one after the other: the bias of a bf16 tile comes into one of two
    places in the LDS by turns while the one before may still be read.  Large integer biases, no two alike in a group, some groups
    without, ragged last columns, K of one chunk and of several: bit for bit, twice."""
    rng = np.random.default_rng(17)
    shapes = [(16, 16, 1000), (32, 16, 900), (5, 208, 770), (20, 272, 1030), (1, 528, 333), (17, 1040, 520), (9, 1040, 1100), (31, 80, 640)]
    specs = []
    for i, (M, K, N) in enumerate(shapes):
        b = (rng.permutation(4 * N)[:N] - 2 * N).astype(np.float32) if i not in (2, 5) else None
        specs.append({"X": rng.integers(-4, 5, (M, K)).astype(np.float32), "W": rng.integers(-3, 4, (K, N)).astype(np.float32),
                      "b": b, "act": "relu" if i % 2 else "none", "s_x": 0.125, "s_w": 0.25})
    G = U.Groups(specs, dtype_name, n_workgroups=8)
    cls = np.where(G.plan.order < 0, -1, G.plan.tiles["cls"][np.maximum(G.plan.order, 0) & 0xFFFFFF]).reshape(-1, 8)
    for c in (0, 1):                                         # classes of 16 and 32 rows
        assert any(np.all(cls[i: i + 4, w] == c) for w in range(8) for i in range(len(cls) - 3)), c
    for rep in range(2):
        for (M, K, N), y, yref in zip(shapes, G.run(), G.expected()):
            assert np.array_equal(y, ref.bf16_decode(ref.bf16_encode(yref))), (dtype_name, rep, M, K, N)


def test_long_k_tiles_visited_in_parts(dtype_name="bf16"):
    """Batches of 17 to 64 rows with K >= 8192 (bf16; fp8 tiles are not split): the launch visits each tile in two
    parts of K whose sums meet in the workspace.  Integer-valued operands make every order of addition exact, so the result must be
    the oracle's bit for bit: ragged K (a part boundary inside a fragment pair, a last fragment cut short),
    ragged rows and columns, next to groups that are not split; twice, on grids of different sizes (who arrives
    last changes), and three times in a row on one plan (the arrival counters return to zero)."""
    rng = np.random.default_rng(17)
    shapes = [(40, 8208, 200), (64, 11024, 136), (17, 8192, 70), (8, 8192, 40), (33, 12304, 24), (64, 4080, 130), (20, 16384, 16)]
    acts = ["relu", "none", "relu", "none", "none", "relu", "none"]
    specs = []
    for (M, K, N), act in zip(shapes, acts):
        X = rng.integers(-4, 5, (M, K)).astype(np.float32)
        W = rng.integers(-3, 4, (K, N)).astype(np.float32)
        b = rng.integers(-8, 9, N).astype(np.float32)
        specs.append({"X": X, "W": W, "b": b, "act": act, "s_x": 0.125, "s_w": 0.25})
    for W_ in (None, 24):
        G = U.Groups(specs, dtype_name, n_workgroups=W_)
        assert G.plan.n_split_tiles > 0
        parts = {int(e >> 28) + 1 for e in G.plan.order if e >= 0}
        assert parts == {1, 2}
        want = [ref.bf16_decode(ref.bf16_encode(y)) for y in G.expected()]
        for rep in range(3):
            for (M, K, N), y, yref in zip(shapes, G.run(), want):
                assert np.array_equal(y, yref), (dtype_name, W_, rep, M, K, N, np.argwhere(y != yref)[:5])
        if dtype_name == "bf16":
            # new activations at the same addresses: the parts that come back from the workspace must be this
            # launch's (the visit that adds them may run on another compute die than the ones that wrote them)
            for i, sp in enumerate(specs):
                G.keep[3 * i].mul_(-2.0)
                G.bits[i]["X"] = casts.bf16_bits(-2.0 * sp["X"])
            want = [ref.bf16_decode(ref.bf16_encode(y)) for y in G.expected()]
            for (M, K, N), y, yref in zip(shapes, G.run(), want):
                assert np.array_equal(y, yref), ("rescaled", W_, M, K, N, np.argwhere(y != yref)[:5])
    # real values: against the oracle at the usual tolerance
    specs = [U.rand_spec(rng, M, K, N, act, bias=True) for (M, K, N), act in zip(shapes, ["gelu_erf", "silu", "none", "relu", "gelu_tanh", "none", "relu"])]
    G = U.Groups(specs, dtype_name)
    for (M, K, N), y, yref in zip(shapes, G.run(), G.expected()):
        assert_close(y, yref, TOL[dtype_name], "split K %s" % ((M, K, N),))


def test_last_round_panel_tiles_visited_in_parts(dtype_name="bf16"):
    """A bf16 launch of panel tiles alone, all of one K: the tiles of the last, partial round are visited in two to four
    parts of K whose raw sums meet in the workspace.  Integer-valued operands make every order of addition exact, so
    the result must be the oracle's bit for bit: ragged rows and columns, a K that is not a multiple of the parts'
    unit, two grid sizes (two and four parts), three calls in a row on one plan (the counters return to zero), and
    (bf16) new activations at the same addresses."""
    rng = np.random.default_rng(19)
    shapes = [(300, 2064, 500), (600, 2064, 300)]
    specs = []
    for (M, K, N), act in zip(shapes, ["relu", "none"]):
        X = rng.integers(-4, 5, (M, K)).astype(np.float32)
        W = rng.integers(-3, 4, (K, N)).astype(np.float32)
        b = rng.integers(-8, 9, N).astype(np.float32)
        specs.append({"X": X, "W": W, "b": b, "act": act, "s_x": 0.125, "s_w": 0.25})
    seen = set()
    for W_ in (8, 24):
        G = U.Groups(specs, dtype_name, n_workgroups=W_)
        assert G.plan.n_panel_split_tiles == 10 % W_ and G.plan.n_split_tiles == 0
        parts = {int(e >> 28) + 1 for e in G.plan.order if e >= 0}
        seen |= parts
        want = [ref.bf16_decode(ref.bf16_encode(y)) for y in G.expected()]
        for rep in range(3):
            for (M, K, N), y, yref in zip(shapes, G.run(), want):
                assert np.array_equal(y, yref), (dtype_name, W_, rep, M, K, N, np.argwhere(y != yref)[:5])
        if dtype_name == "bf16":
            for i, sp in enumerate(specs):
                G.keep[3 * i].mul_(-2.0)
                G.bits[i]["X"] = casts.bf16_bits(-2.0 * sp["X"])
            want = [ref.bf16_decode(ref.bf16_encode(y)) for y in G.expected()]
            for (M, K, N), y, yref in zip(shapes, G.run(), want):
                assert np.array_equal(y, yref), ("rescaled", W_, M, K, N, np.argwhere(y != yref)[:5])
    assert seen == {1, 2, 4}
    # tiles of one launch in three and in four parts (two parts per workgroup on average)
    shapes = [(900, 4112, 300), (600, 4112, 300)]
    specs = []
    for M, K, N in shapes:
        X = rng.integers(-3, 4, (M, K)).astype(np.float32)
        W = rng.integers(-3, 4, (K, N)).astype(np.float32)
        specs.append({"X": X, "W": W, "b": rng.integers(-8, 9, N).astype(np.float32), "act": "none", "s_x": 0.125, "s_w": 0.25})
    G = U.Groups(specs, dtype_name, n_workgroups=24)
    assert G.plan.n_panel_split_tiles == 14 and {int(e >> 28) + 1 for e in G.plan.order if e >= 0} == {3, 4}
    want = [ref.bf16_decode(ref.bf16_encode(y)) for y in G.expected()]
    for rep in range(2):
        for (M, K, N), y, yref in zip(shapes, G.run(), want):
            assert np.array_equal(y, yref), ("mixed parts", rep, M, K, N, np.argwhere(y != yref)[:5])
    shapes = [(300, 2064, 500), (600, 2064, 300)]
    specs = [U.rand_spec(rng, M, K, N, act, bias=True) for (M, K, N), act in zip(shapes, ["gelu_erf", "silu"])]
    G = U.Groups(specs, dtype_name, n_workgroups=8)
    for (M, K, N), y, yref in zip(shapes, G.run(), G.expected()):
        assert_close(y, yref, TOL[dtype_name], "panel split K %s" % ((M, K, N),))


def test_fp32_tiles_at_the_edges_of_their_range():
    """fp32 tiles: row blocks just below and above 16 and 64, K shorter than, equal to and beyond one piece per wave, rows
    and columns whose 16-byte pieces are not aligned.  Integer-valued operands: bit for bit; real ones: 1e-5 (the sums of
    at most 1000 products carry about sqrt(1000) 2^-24 = 2e-6)."""
    rng = np.random.default_rng(29)
    shapes = [(1, 1, 1), (15, 3, 3), (16, 16, 64), (16, 256, 66), (17, 17, 10), (33, 64, 63), (63, 255, 130), (64, 257, 64), (65, 1000, 128),
              (4, 512, 512), (200, 260, 68), (48, 4, 200), (16, 270, 12)]
    for integers in (True, False):
        specs = []
        for M, K, N in shapes:
            sp = U.rand_spec(rng, M, K, N, "relu" if M % 2 else "none", bias=N != 64)
            if integers:
                sp["X"], sp["W"] = np.round(4 * sp["X"]), np.round(4 * sp["W"] * np.sqrt(K)).astype(np.float32)
                sp["b"] = None if sp["b"] is None else np.round(800 * sp["b"])
            specs.append(sp)
        G = U.Groups(specs, "f32")
        for (M, K, N), y, yref in zip(shapes, G.run(), G.expected()):
            if integers:
                assert np.array_equal(y, yref), (M, K, N)
            else:
                assert_close(y, yref, TOL["f32"], "fp32 %s" % ((M, K, N),))


@pytest.mark.parametrize("dtype_name,out_name", [("bf16", None), ("fp8", None), ("fp8", "fp8")])
def test_block_tiles_at_the_edges_of_their_range(dtype_name, out_name):
    """Launches planned with block tiles (128 x 128): one to four row fragments, rows just below and above a tile, columns
    that leave a wave idle or cut a 16-byte piece short, K from one chunk through every place of the four-pair ring.
    Integer-valued operands make every order of addition exact: bf16 outputs must be the oracle's bit for bit, twice."""
    rng = np.random.default_rng(23)
    k = 1 if dtype_name == "bf16" else 2
    shapes = [(65, 16, 10), (96, 64 * k, 128), (97, 72 * k, 130), (128, 128 * k, 200), (129, 136 * k, 72), (160, 256 * k, 127), (200, 272 * k, 264),
              (31, 384 * k, 64), (1, 520 * k, 33), (300, 768 * k, 16), (64, 1040 * k, 136), (33, 896 * k, 8)]
    acts = ["relu", "none"] * 6
    specs = []
    for (M, K, N), act in zip(shapes, acts):
        specs.append({"X": rng.integers(-4, 5, (M, K)).astype(np.float32), "W": rng.integers(-3, 4, (K, N)).astype(np.float32),
                      "b": rng.integers(-8, 9, N).astype(np.float32), "act": act, "s_x": 0.125, "s_w": 0.25})
    G = U.Groups(specs, dtype_name, out_dtype_name=out_name)
    assert [int(v) for v in G.plan.classes[-1]][1:3] == [128, 128]        # next to streaming tiles for the batches up to 64 rows
    for rep in range(2):
        for (M, K, N), y, yref in zip(shapes, G.run(), G.expected()):
            if out_name is None:
                assert np.array_equal(y, ref.bf16_decode(ref.bf16_encode(yref))), (dtype_name, rep, M, K, N)
            else:
                assert np.array_equal(y, ref.e4m3_decode(ref.e4m3_encode(yref, 1.0), 1.0)), (dtype_name, rep, M, K, N)
    specs = [U.rand_spec(rng, M, K, N, act, bias=i % 2 == 0) for i, ((M, K, N), act) in
             enumerate(zip(shapes, ["gelu_erf", "silu", "none", "relu", "gelu_tanh", "none"] * 2))]
    G = U.Groups(specs, dtype_name)
    for (M, K, N), y, yref in zip(shapes, G.run(), G.expected()):
        assert_close(y, yref, TOL[dtype_name], "block tiles %s" % ((M, K, N),))


@pytest.mark.parametrize("dtype_name", ["bf16", "fp8"])
def test_block_tiles_visited_in_parts(dtype_name):
    """Block tiles of a long K: every number of parts (by the number of tiles of the launch; fp8 tiles are not split), parts that cover two pairs only
    and ones that go round the ring, ragged K, rows and columns, next to a streaming batch that is split itself.
    Integer-valued operands: bit for bit, three calls in a row (the counters return to zero), then new activations at
    the same addresses (a part of an earlier call must not be read)."""
    rng = np.random.default_rng(31)
    seen = set()
    for shapes in ([(75, 1040, 130), (130, 2064, 200), (200, 4112, 72), (40, 8208, 136), (66, 512, 40)],
                   [(300, 1552, 264), (97, 1024, 17)], [(1100, 3088, 1290)], [(600, 4112, 1900)]):
        specs = []
        for M, K, N in shapes:
            specs.append({"X": rng.integers(-3, 4, (M, K)).astype(np.float32), "W": rng.integers(-2, 3, (K, N)).astype(np.float32),
                          "b": rng.integers(-8, 9, N).astype(np.float32), "act": "relu" if M % 2 else "none", "s_x": 0.125, "s_w": 0.25})
        G = U.Groups(specs, dtype_name)
        assert int(G.plan.classes[-1][1]) == 128
        seen |= {int(e >> 28) + 1 for e in G.plan.order if e >= 0 and G.plan.tiles[e & 0xFFFFFF]["cls"] == 3}
        want = [ref.bf16_decode(ref.bf16_encode(y)) for y in G.expected()]
        for rep in range(3):
            for (M, K, N), y, yref in zip(shapes, G.run(), want):
                assert np.array_equal(y, yref), (dtype_name, rep, M, K, N)
        if dtype_name == "bf16":
            for i, sp in enumerate(specs):
                G.keep[3 * i].mul_(-2.0)
                G.bits[i]["X"] = casts.bf16_bits(-2.0 * sp["X"])
            for (M, K, N), y, yref in zip(shapes, G.run(), [ref.bf16_decode(ref.bf16_encode(y)) for y in G.expected()]):
                assert np.array_equal(y, yref), ("rescaled", M, K, N)
    assert seen == ({1, 2, 3, 4} if dtype_name == "bf16" else {1})


def test_block_tiles_in_parts_without_a_workspace_are_still_computed():
    """An order with parts in a launch that states no split tiles: the first visit of a tile multiplies the whole K."""
    rng = np.random.default_rng(41)
    specs = [{"X": rng.integers(-3, 4, (M, K)).astype(np.float32), "W": rng.integers(-2, 3, (K, N)).astype(np.float32),
              "b": rng.integers(-8, 9, N).astype(np.float32), "act": "none"} for M, K, N in ((100, 1040, 200), (300, 2064, 72))]
    G = U.Groups(specs, "bf16")
    assert int(G.plan.classes[-1][1]) == 128 and G.plan.n_split_tiles == 0 and max(int(e >> 28) for e in G.plan.order if e >= 0) > 0
    G.plan.c.n_panel_split_tiles, G.plan.c.d_workspace, G.plan.c.workspace_bytes = 0, None, 0
    for y, yref in zip(G.run(), G.expected()):
        assert np.array_equal(y, ref.bf16_decode(ref.bf16_encode(yref)))


@pytest.mark.parametrize("shapes,W_", [([(300, 2064, 500), (600, 2064, 300)], 8), ([(40, 8208, 200), (17, 8192, 70)], None),
                                       ([(75, 1040, 130), (200, 4112, 72), (40, 8208, 136)], None)])
def test_only_the_counters_of_a_workspace_have_to_be_zero(shapes, W_):
    """Panel, streaming and block tiles in parts on a workspace whose partial sums start as NaN: bit for bit."""
    rng = np.random.default_rng(59)
    specs = [{"X": rng.integers(-3, 4, (M, K)).astype(np.float32), "W": rng.integers(-2, 3, (K, N)).astype(np.float32),
              "b": None, "act": "none"} for M, K, N in shapes]
    G = U.Groups(specs, "bf16", n_workgroups=W_)
    counters = 4 * (G.plan.n_split_tiles + G.plan.n_panel_split_tiles)
    assert counters > 0
    G.plan.d_workspace.fill_(255)
    B.epara_workspace_init(G.plan.d_workspace.data_ptr(), -(-counters // 256) * 256, R.current_stream_handle())
    for sh, y, yref in zip(shapes, G.run(), G.expected()):
        assert np.array_equal(y, ref.bf16_decode(ref.bf16_encode(yref))), sh


def test_two_plans_of_one_argument_array_do_not_disturb_each_other():
    """The split tiles of a plan meet at places of its own: making a second plan, for another grid, from the same array of
    arguments changes neither the array nor the first plan."""
    rng = np.random.default_rng(53)
    specs = [{"X": rng.integers(-3, 4, (M, K)).astype(np.float32), "W": rng.integers(-2, 3, (K, N)).astype(np.float32),
              "b": None, "act": "none"} for M, K, N in ((75, 1040, 130), (200, 4112, 72), (40, 8208, 136))]
    G = U.Groups(specs, "bf16")
    before = G.args.copy()
    plans = [R.LaunchPlan(G.args, B.EPARA_BF16, U.DEV, W) for W in (256, 120, 256)]
    assert plans[0].workspace_bytes and plans[1].workspace_bytes and plans[0].args["reserved"].tolist() != plans[1].args["reserved"].tolist()
    assert np.array_equal(G.args, before)
    want = [ref.bf16_decode(ref.bf16_encode(y)) for y in G.expected()]
    for plan in (plans[0], plans[1], plans[2], plans[0]):
        for y in G.Y:
            y.zero_()
        R.grouped_forward(plan, B.EPARA_BF16)
        torch.cuda.synchronize()
        for y, w in zip(G.Y, want):
            assert np.array_equal(U.fetch(y), w)


def test_launches_with_split_tiles_take_turns_on_one_workspace():
    """Panel tiles in four parts, streaming tiles in two, block tiles in parts and both kinds in one launch, all on one
    workspace that is zeroed once: the counters lie in front of every launch's partial sums, so each launch finds its own
    at zero whatever ran before it.  Integer-valued operands: bit for bit, in three different orders."""
    rng = np.random.default_rng(37)
    groups = []
    for shapes, W_, kind in (([(300, 2064, 500), (600, 2064, 300)], 8, 256), ([(40, 8208, 200), (17, 8192, 70)], None, None),
                             ([(300, 1552, 264), (97, 1024, 17)], None, 128), ([(75, 1040, 130), (200, 4112, 72), (40, 8208, 136)], None, 128)):
        specs = [{"X": rng.integers(-3, 4, (M, K)).astype(np.float32), "W": rng.integers(-2, 3, (K, N)).astype(np.float32),
                  "b": rng.integers(-8, 9, N).astype(np.float32), "act": "relu" if M % 2 else "none"} for M, K, N in shapes]
        G = U.Groups(specs, "bf16", n_workgroups=W_)
        assert kind is None or int(G.plan.classes[-1][1]) == kind
        assert 0 < G.plan.n_split_tiles + G.plan.n_panel_split_tiles <= 64          # as many counters as share a workspace
        assert max(int(e >> 28) + 1 for e in G.plan.order if e >= 0) == (2 if kind is None else 4)
        groups.append((shapes, G, [ref.bf16_decode(ref.bf16_encode(y)) for y in G.expected()]))
    ws = torch.empty(max(G.plan.workspace_bytes for _, G, _ in groups), dtype=torch.uint8, device=U.DEV)
    B.epara_workspace_init(ws.data_ptr(), ws.numel(), R.current_stream_handle())
    for _, G, _ in groups:
        G.plan.c.d_workspace, G.plan.c.workspace_bytes = ws.data_ptr(), ws.numel()
    for turn in ([0, 2, 1, 3], [3, 0, 3, 2], [2, 1, 0, 2, 3, 0]):
        for i in turn:
            shapes, G, want = groups[i]
            for sh, y, yref in zip(shapes, G.run(), want):
                assert np.array_equal(y, yref), (turn, i, sh)


@pytest.mark.parametrize("dtype_name", ["bf16", "fp8"])
@pytest.mark.parametrize("rows,d,ffn", [([3, 40, 300], 128, 352), ([20, 200], 256, 8224), ([70, 200], 2064, 80), ([75, 130, 237], 272, 208), ([97, 1], 48, 80)])
def test_gated_block_tiles(dtype_name, rows, d, ffn):
    mix = make_mix(4, d=d, ffn=ffn, rows=rows)
    staged = StagedMix(mix, dtype_name, U.DEV, s_h=[1.0] * len(rows) if dtype_name == "fp8" else None)
    assert int(staged.plans()[-1].classes[-1][1]) == 128 and (ffn > 8192 or int(staged.plans()[0].classes[-1][1]) == 128)
    check_mix(mix, dtype_name)


def test_identity_zero_and_ones_weights_bf16():
    rng = np.random.default_rng(12)
    X = rng.standard_normal((37, 64)).astype(np.float32)
    b = (rng.standard_normal(64) * 0.5).astype(np.float32)
    specs = [{"X": X, "W": np.eye(64, dtype=np.float32), "b": b, "act": "none"},
             {"X": X, "W": np.zeros((64, 48), dtype=np.float32), "b": b[:48], "act": "gelu_erf"},
             {"X": np.round(X * 4) / 4, "W": np.ones((64, 20), dtype=np.float32), "b": None, "act": "none"}]
    G = U.Groups(specs, "bf16")
    y, want = G.run(), G.expected()
    Xb = ref.bf16_decode(G.bits[0]["X"])
    assert np.array_equal(y[0], ref.bf16_decode(ref.bf16_encode(Xb + b.astype(np.float64))))
    assert_close(y[1], want[1], TOL["bf16"], "zero weights")
    assert np.all(y[1] == y[1][0])                                   # act(b) broadcast over rows
    assert_close(y[2], want[2], TOL["bf16"], "ones weights")


@pytest.mark.parametrize("dtype_name", ["f32", "bf16"])
def test_linearity_in_x(dtype_name):
    rng = np.random.default_rng(13)
    M, K, N = 90, 128, 72
    X1, X2 = rng.standard_normal((M, K)).astype(np.float32), rng.standard_normal((M, K)).astype(np.float32)
    W = (rng.standard_normal((K, N)) / np.sqrt(K)).astype(np.float32)
    a, c = 1.75, -0.375
    f = lambda X: U.Groups([{"X": X, "W": W, "b": None, "act": "none"}], dtype_name).run()[0]
    lhs, rhs = f(a * X1 + c * X2), a * f(X1) + c * f(X2)
    assert_close(lhs, rhs, 3 * TOL[dtype_name], "linearity")


@pytest.mark.parametrize("shapes", [[(3, 20, 64 * 42)], [(3, 20, 64 * 43)], [(2, 24, 12)] * 14, [(2, 24, 12)] * 15])
def test_fp32_launches_around_the_tables_that_are_read_ahead(shapes):
    """Launches whose tables of tiles (42 x 24 bytes) or arguments (14 x 72 bytes) just fit what a workgroup asks for ahead, and the next ones."""
    rng = np.random.default_rng(22)
    G = U.Groups([U.rand_spec(rng, M, K, N) for M, K, N in shapes], "f32")
    for y, yref in zip(G.run(), G.expected()):
        assert_close(y, yref, TOL["f32"], "fp32 tables %d" % len(shapes))


def test_fp32_small_batches_with_awkward_shapes():
    """Batches of at most 16 rows take the fp32 path that cuts K into sixteen shares of pieces of 16: K of less than a
    piece, of fewer pieces than shares, not a multiple of a piece, ragged column tiles, every activation, next to a group of
    the 64-row class in the same launch."""
    rng = np.random.default_rng(21)
    acts = ["none", "relu", "gelu_erf", "gelu_tanh", "silu"]
    shapes = [(1, 1, 1), (7, 3, 10), (16, 7, 65), (3, 17, 130), (16, 100, 64), (9, 513, 77), (2, 2048, 5), (40, 33, 70), (16, 64, 128)]
    specs = [U.rand_spec(rng, M, K, N, acts[i % len(acts)], bias=i % 3 != 0) for i, (M, K, N) in enumerate(shapes)]
    G = U.Groups(specs, "f32")
    assert sorted(set(int(c) for c in G.plan.tiles["cls"])) == [0, 1]
    for (M, K, N), y, yref in zip(shapes, G.run(), G.expected()):
        assert_close(y, yref, TOL["f32"], "fp32 small %s" % ((M, K, N),))
    # and the same values whatever the grid size (fixed summation order)
    y_a = U.Groups(specs, "f32", n_workgroups=8).run()
    y_b = U.Groups(specs, "f32", n_workgroups=256).run()
    for a, b in zip(y_a, y_b):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("M,K", [(16, 256), (16, 1024), (64, 256), (64, 1024), (200, 4096)])
def test_fp32_error_against_64_bits(M, K):
    """fp32 tiles add K in sixteen (64 rows: eight) shares, so the error is that of sums of n = K / 16 (K / 8) products: a
    rounding errs by about 0.4 u (u = 2^-24) of a partial sum that grows like the root of its length, 0.4 sqrt(n / 2) u = 0.29 sqrt(n) u in all,
    and adding the shares by another u.  Bound: (0.33 sqrt(n) + 1.2) u, below what one sum over K shows (64 rows, K = 1024:
    5.7e-7, here 2.1e-7, bound 2.9e-7)."""
    rng = np.random.default_rng(61)
    X = rng.uniform(-1, 1, (M, K)).astype(np.float32)
    W = (rng.standard_normal((K, 512)) / np.sqrt(K)).astype(np.float32)
    y = U.Groups([{"X": X, "W": W, "b": None, "act": "none"}], "f32").run()[0]
    want = X.astype(np.float64) @ W.astype(np.float64)
    n = K / (16 if M <= 16 else 8)
    assert np.linalg.norm(y - want) <= (0.33 * np.sqrt(n) + 1.2) * 2.0 ** -24 * np.linalg.norm(want)


# ---- independence and determinism ------------------------------------------------------------------

def test_group_order_row_order_and_grid_size_do_not_change_a_single_bit():
    rng = np.random.default_rng(14)
    shapes = [(3, 256, 96, "gelu_erf"), (300, 128, 260, "relu"), (64, 512, 64, "none"), (17, 64, 10, "silu"), (700, 96, 300, "none")]
    specs = [U.rand_spec(rng, M, K, N, act) for M, K, N, act in shapes]
    base = U.Groups(specs, "bf16")
    y0 = base.run()
    raw0 = [t.view(torch.int16).cpu().numpy() for t in base.raw()]
    perm = [3, 0, 4, 2, 1]
    y1 = U.Groups([specs[i] for i in perm], "bf16").run()
    for j, i in enumerate(perm):
        assert np.array_equal(y1[j], y0[i])
    for W in (8, 64, 128):
        g = U.Groups(specs, "bf16", n_workgroups=W)
        g.run()
        for a, t in zip(raw0, g.raw()):
            assert np.array_equal(a, t.view(torch.int16).cpu().numpy())
    # permuting the rows of X permutes the rows of Y; splitting a batch in two reproduces the same rows
    p = rng.permutation(300)
    s = dict(specs[1]); s["X"] = specs[1]["X"][p]
    top, bottom = dict(specs[1]), dict(specs[1])
    top["X"], bottom["X"] = specs[1]["X"][:100], specs[1]["X"][100:]
    ys = U.Groups([s, top, bottom], "bf16").run()
    assert np.array_equal(ys[0], y0[1][p])
    assert_close(np.vstack([ys[1], ys[2]]), y0[1], 1e-2, "split batch")   # tile classes differ: not bitwise
    # run to run
    again = base.run()
    for a, b in zip(y0, again):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("dtype_name", ["bf16", "fp8"])
def test_gated_and_fp8_outputs_do_not_depend_on_the_grid_or_the_other_services(dtype_name):
    """SwiGLU services in block tiles (256 workgroups) and in panel tiles (fewer than 128), all of them or one alone, K long
    enough to be split and of more pairs of stages than the rings hold: the hidden activations (gated), and for fp8 the
    outputs of the down launch, are the same bits."""
    import copy
    mix = make_mix(4, d=1200, ffn=2416, rows=[75, 130, 40, 300])
    s_h = [0.02] * 4 if dtype_name == "fp8" else None
    base = StagedMix(mix, dtype_name, U.DEV, s_h=s_h)
    assert int(base.plans()[0].classes[-1][1]) == 128 and (dtype_name == "bf16" or int(base.plans()[1].classes[-1][1]) == 128)

    def bits(staged):
        staged.run()
        torch.cuda.synchronize()
        return {(g, label): t.view(torch.uint8).cpu().numpy() for launch in staged.outputs[0] for g, label, t in launch
                if label == "H" or dtype_name == "fp8"}
    want = bits(base)
    assert len(want) == (8 if dtype_name == "fp8" else 4)
    for W in (64, 120, 128):
        got = bits(StagedMix(mix, dtype_name, U.DEV, s_h=s_h, n_workgroups=W, host_bits=base.host_bits))
        for key in want:
            assert np.array_equal(got[key], want[key]), (W, key)
    for g in range(4):
        alone = copy.copy(mix)
        alone.services = mix.services[g: g + 1]
        got = bits(StagedMix(alone, dtype_name, U.DEV, s_h=None if s_h is None else s_h[:1], host_bits=base.host_bits[g: g + 1]))
        for (_, label), b in got.items():
            assert np.array_equal(b, want[g, label]), (g, label)


# ---- edge cases -------------------------------------------------------------------------------------

@pytest.mark.parametrize("dtype_name,tiles", [("f32", None), ("bf16", "block"), ("bf16", "panel"), ("fp8", "block"), ("fp8", "panel")])
def test_ragged_and_degenerate_groups(dtype_name, tiles):
    rng = np.random.default_rng(15)
    kmul = 16 if dtype_name == "fp8" else 8
    shapes = [(0, 64, 32, "none"), (1, kmul, 1, "none"), (1, 64, 10, "relu"), (64, 5 * kmul, 33, "gelu_erf"),
              (65, 3 * kmul, 31, "silu"), (255, 7 * kmul, 255, "gelu_tanh"), (256, 128, 256, "none"),
              (257, 64 + kmul, 257, "relu"), (0, 32, 8, "none"), (513, 2 * kmul, 7, "none")]
    specs = [U.rand_spec(rng, M, K, N, act) for M, K, N, act in shapes]
    G = tall_groups(specs, dtype_name, tiles)
    got, want = G.run(), G.expected()
    for sh, y, yref in zip(shapes, got, want):
        assert y.shape == yref.shape
        if y.size:
            assert_close(y, yref, TOL[dtype_name], str(sh))


@pytest.mark.parametrize("tiles", ["panel", "block"])
@pytest.mark.parametrize("dtype_name", ["bf16", "fp8"])
def test_every_activation_on_whole_and_ragged_tall_tiles(dtype_name, tiles):
    """The matrix-core kernels use the hardware's exp / reciprocal and a rational erf in their epilogue; whole 256 x 256
    tiles run an unrolled epilogue, ragged ones a loop, block tiles one of their own: all against the fp64 oracle, with
    bias, K of one to five stages incl. an odd stage count and a ragged last stage."""
    rng = np.random.default_rng(16)
    kmul = 16 if dtype_name == "fp8" else 8
    acts = ["none", "relu", "gelu_erf", "gelu_tanh", "silu"]
    shapes = [(512, 24 * kmul, 512, acts[i % 5]) if i < 5 else (300, (4 * i + 1) * kmul, 520, acts[i % 5]) for i in range(10)]
    specs = [U.rand_spec(rng, M, K, N, act) for M, K, N, act in shapes]
    for sp in specs:                                                     # activations need arguments of both signs and sizes
        sp["X"] *= 2.0
    G = tall_groups(specs, dtype_name, tiles)
    got, want = G.run(), G.expected()
    for sh, y, yref in zip(shapes, got, want):
        assert_close(y, yref, TOL[dtype_name], str(sh))


@pytest.mark.parametrize("tiles", ["panel", "block"])
def test_output_beyond_four_gibibytes_is_addressed_with_64_bits(tiles):
    """One group whose output has more than 2^32 bytes (and its last rows more than 2^31 elements in): rows
    sampled from the start, the 4 GiB boundary and the end against the oracle, tiles whole and ragged."""
    rng = np.random.default_rng(17)
    M, K, N = 36100, 16, 60040
    sp = U.rand_spec(rng, M, K, N, "relu")
    xb, wb = casts.bf16_bits(sp["X"]), casts.bf16_bits(sp["W"])
    dX = R.device_tensor_from_bits(xb, B.EPARA_BF16, U.DEV)
    dW = R.pack_weights(R.device_tensor_from_bits(wb, B.EPARA_BF16, U.DEV), B.EPARA_BF16)
    db = torch.from_numpy(sp["b"]).to(U.DEV)
    dY = torch.zeros((M, N), dtype=torch.bfloat16, device=U.DEV)
    assert dY.numel() * 2 > 2 ** 32
    plan = R.LaunchPlan(np.array([R.group_args(dX, dW, dY, M, K, N, "relu", bias=db)], dtype=B.GROUP_ARGS), B.EPARA_BF16, U.DEV,
                        TALL[tiles][0])
    assert int(plan.classes[-1][1]) == TALL[tiles][1]
    R.grouped_forward(plan, B.EPARA_BF16)
    torch.cuda.synchronize()
    edge = 2 ** 32 // (2 * N)                                            # the row that straddles byte 2^32
    rows = sorted({0, 1, 255, 256, edge - 1, edge, edge + 1, 2 ** 31 // N, 2 ** 31 // N + 1, M - 257, M - 2, M - 1}
                  | set(int(r) for r in rng.integers(0, M, 12)))
    got = dY[torch.tensor(rows, device=U.DEV)].float().cpu().numpy()
    want = ref.dense_forward(ref.bf16_decode(xb[rows]), ref.bf16_decode(wb), sp["b"], "relu")
    assert_close(got, want, TOL["bf16"], "rows around the 4 GiB boundary")
    # nothing outside the group's rows x columns was touched: the padding rows of the last tile row stay unwritten
    assert torch.count_nonzero(dY[M - 1]).item() > 0
    del dY
    torch.cuda.empty_cache()


def test_nothing_to_do_is_ok():
    G = U.Groups([], "bf16")
    assert G.run() == []
    rng = np.random.default_rng(16)
    G = U.Groups([U.rand_spec(rng, 0, 64, 32), U.rand_spec(rng, 0, 32, 8)], "bf16")
    assert [y.shape for y in G.run()] == [(0, 32), (0, 8)]


def test_every_activation_fp32():
    rng = np.random.default_rng(17)
    specs = [U.rand_spec(rng, 33, 100, 70, act, x_uniform=True) for act in ("none", "relu", "gelu_erf", "gelu_tanh", "silu")]
    for s in specs:
        s["X"] = s["X"] * 3
    G = U.Groups(specs, "f32")
    for s, y, yref in zip(specs, G.run(), G.expected()):
        assert_close(y, yref, TOL["f32"], s["act"])


def test_pack_weights_layout_round_trip():
    # packed fragment (nb, ks), chunk q*16+r holds W[ks*32 + 8q .. +7][nb*16 + r] (bf16), zero padded; the
    # stages of a column block are padded to a multiple of four
    rng = np.random.default_rng(18)
    K, N = 72, 37
    bits = rng.integers(1, 2 ** 15, (K, N)).astype(np.uint16)
    W = R.device_tensor_from_bits(bits, B.EPARA_BF16, U.DEV)
    P = R.pack_weights(W, B.EPARA_BF16)
    torch.cuda.synchronize()
    p = P.cpu().numpy().view(np.uint16).reshape(3, 4, 4, 16, 8)          # [nb][ks][q][r][e]
    want = np.zeros((3, 4, 4, 16, 8), dtype=np.uint16)
    for nb in range(3):
        for ks in range(3):
            for q in range(4):
                for r in range(16):
                    for e in range(8):
                        k, n = ks * 32 + q * 8 + e, nb * 16 + r
                        if k < K and n < N:
                            want[nb, ks, q, r, e] = bits[k, n]
    assert np.array_equal(p, want)


# ---- what the kernel reads is what the reference planner wrote ----------------------------------------

@pytest.mark.parametrize("index,shrink", [(4, {}), (3, {}), (2, {})])
def test_device_copies_of_the_tile_table_and_visit_order_are_the_reference_planners(index, shrink):
    from oracle import planner as P
    staged = StagedMix(make_mix(index, **shrink), None, U.DEV)
    for plan in staged.plans():
        tiles = plan.d_tiles.cpu().numpy()[: plan.tiles.nbytes].view(B.TILE)
        order = plan.d_order.cpu().numpy()[: plan.order.nbytes].view(np.int32)
        args = plan.d_args.cpu().numpy()[: plan.args.nbytes].view(B.GROUP_ARGS)
        assert np.array_equal(args, plan.args)
        gated = bool(np.all(plan.args["act"] == B.EPARA_ACT_SWIGLU))
        groups = [(int(a["M"]), int(a["K"]), int(a["N"])) + ((True,) if gated else ()) for a in plan.args]
        classes = [tuple(int(v) for v in c) for c in plan.classes]
        row_off, x_off, y_off, want_tiles = P.plan_groups([g[:3] for g in groups], classes)
        assert [tuple(int(v) for v in t) for t in tiles] == want_tiles
        want_order = P.schedule_tiles(groups, classes, plan.n_stream_classes, want_tiles, plan.n_workgroups, 8, 1, 4)
        assert order.tolist() == want_order
        assert plan.row_off.tolist() == row_off and plan.x_off.tolist() == x_off and plan.y_off.tolist() == y_off


def test_end_to_end_error_against_the_unrounded_masters_is_reported():
    """Informative: the parity gate compares against an oracle fed the same rounded inputs; this is the error
    against the fp32 masters, i.e. including the storage formats' own rounding (bf16: about 2^-9 per operand)."""
    mix = make_mix(4, d=512, ffn=1376)
    staged = StagedMix(mix, "bf16", U.DEV)
    staged.run()
    torch.cuda.synchronize()
    from parity_util import rel_err
    worst = 0.0
    for (g, label, Y) in staged.results()[-1]:
        svc = mix.services[g]
        _H, Yref = ref.ffn_swiglu(svc.X.astype(np.float64), svc.Wgate.astype(np.float64), svc.Wup.astype(np.float64), svc.Wdown.astype(np.float64))
        worst = max(worst, rel_err(Y, Yref))
    print("end-to-end max relative error vs fp32 masters (bf16 decode FFN, reduced): %.3e" % worst)
    assert worst < 5e-2


# ---- the five mixes ---------------------------------------------------------------------------------

def test_mix1_mlp_fp32_full():
    check_mix(make_mix(1), "f32")


def test_mix2_small_models_bf16_full():
    check_mix(make_mix(2), "bf16")


def test_mix3_vit_reduced_all_rows():
    check_mix(make_mix(3, images=[2, 1, 1, 3, 1, 2, 1, 1], d=192, ffn=768, tokens=197), "bf16")


def test_mix3_vit_full_size_all_rows():
    check_mix(make_mix(3), "bf16")


def test_mix4_decode_reduced_all_rows():
    check_mix(make_mix(4, d=512, ffn=1376), "bf16")


def test_mix4_decode_fp8_reduced_all_rows():
    # the weight-streaming classes with E4M3 inputs and E4M3 hidden activations (static scale from the oracle)
    check_mix(make_mix(4, d=1024, ffn=2752), "fp8")


def test_mix4_decode_full_size():
    check_mix(make_mix(4), "bf16")


def test_mix4_decode_fp8_full_size():
    check_mix(make_mix(4), "fp8")


@pytest.mark.parametrize("dtype_name", ["bf16", "fp8"])
def test_mix5_prefill_reduced_all_rows(dtype_name):
    check_mix(make_mix(5, d=640, ffn=1664, total_rows=900, len_lo=60, len_hi=300), dtype_name)


@pytest.fixture(scope="module")
def mix5():
    return make_mix(5)


@pytest.mark.parametrize("dtype_name", ["bf16", "fp8"])
def test_mix5_prefill_full_size_all_rows(mix5, dtype_name):
    """Every output element of the 8192-row prefill mix against the fp64 oracle (about a minute of oracle time
    per dtype on the host cores)."""
    check_mix(mix5, dtype_name)


# ---- panel tiles in halves ---------------------------------------------------------------------

@pytest.mark.parametrize("gated", [False, True])
def test_panel_tiles_in_halves_give_the_bits_of_whole_ones(gated):
    """bf16 launches of panel tiles multiply them in halves unless some K is above 2560 (gated 1536): the same groups alone and next to one such group give the
    same bits, those of the fp64 oracle, as all sums are of small integers.  Row counts around the halves' fragments of 32 and around 128 and 256, so that
    a half is missing, of one row or ragged; K of one pair of stages, of several and ragged; whole and ragged columns; with bias and without; a grid small
    enough that a workgroup visits halves of several groups in a row."""
    rng = np.random.default_rng(23)
    limit = 1536 if gated else 2560
    shapes = [(65, 8, 300), (96, 136, 256), (128, 64, 33), (129, 776, 520), (160, 256, 264), (161, 264, 512), (225, 384, 130), (256, 128, 256),
              (257, 192, 257), (290, 320, 10), (384, 768, 384), (385, limit, 300), (512, 200, 700)]
    keep, outs, want = [], [], []
    def stage(M, K, N, i):
        X = rng.integers(-2, 3, (M, K)).astype(np.float32)
        Ws = [rng.integers(-1, 2, (K, N)).astype(np.float32) for _ in range(2 if gated else 1)]
        b = None if gated or i % 3 == 2 else rng.integers(-8, 9, N).astype(np.float32)
        dX = R.device_tensor_from_bits(casts.bf16_bits(X), B.EPARA_BF16, U.DEV)
        dW = [R.pack_weights(R.device_tensor_from_bits(casts.bf16_bits(W), B.EPARA_BF16, U.DEV), B.EPARA_BF16) for W in Ws]
        db = None if b is None else torch.from_numpy(b).to(U.DEV)
        dY = torch.zeros((M, N), dtype=torch.bfloat16, device=U.DEV)
        keep.extend([dX, db] + dW)
        outs.append(dY)
        if gated:
            z, u = X.astype(np.float64) @ Ws[0], X.astype(np.float64) @ Ws[1]
            want.append(z / (1 + np.exp(-z)) * u)
            return R.group_args(dX, dW[0], dY, M, K, N, "swiglu", W2=dW[1])
        want.append(ref.dense_forward(X.astype(np.float64), Ws[0].astype(np.float64), b, "relu"))
        return R.group_args(dX, dW[0], dY, M, K, N, "relu", bias=db)
    args = [stage(M, K, N, i) for i, (M, K, N) in enumerate(shapes)]
    long = stage(70, limit + 8, 40, 0)
    bits = []
    for n_workgroups, groups in ((16, args), (64, args), (16, args + [long])):
        plan = R.LaunchPlan(np.array(groups, dtype=B.GROUP_ARGS), B.EPARA_BF16, U.DEV, n_workgroups)
        assert int(plan.classes[-1][1]) == 256 and plan.n_panel_split_tiles == 0
        for rep in range(2):
            for y in outs:
                y.fill_(float("nan"))
            R.grouped_forward(plan, B.EPARA_BF16)
            torch.cuda.synchronize()
        bits.append([y.view(torch.int16).clone() for y in outs[:len(shapes)]])
    for sh, half, half64, whole, y, w in zip(shapes, *bits, outs, want):
        assert torch.equal(half, whole) and torch.equal(half64, whole), sh
        if gated:
            assert_close(U.fetch(y), w, TOL["bf16"], str(sh))
        else:
            assert np.array_equal(U.fetch(y), ref.bf16_decode(ref.bf16_encode(w))), sh


# ---- the last round of panel tiles in quarters --------------------------------------------------

@pytest.mark.parametrize("dtype_name,gated", [("bf16", True), ("fp8", True), ("fp8", False)])
def test_panel_tiles_of_a_last_round_in_quarters_give_the_bits_of_whole_ones(dtype_name, gated):
    """Launches of panel tiles of one K with a few tiles more than whole rounds multiply those in quarters; the same groups next to one of another K do
    not.  All sums are of small integers: the same bits, the oracle's.  The last tiles have a single row or column, one quarter, ragged ones or four
    whole ones; one and two whole rounds, one tile left to three eighths of a round; K of one pair of stages, ragged, and beyond what is multiplied in halves."""
    rng = np.random.default_rng(29)
    W_, dt, u = 16, B.DTYPE_BY_NAME[dtype_name], 128 if gated else 256
    launches = [[(257, 1552, 8 * u + 5)], [(600, 1552, 5 * u + u // 2 + 3), (130, 1552, 2 * u)], [(400, 2048, 8 * u), (100, 2048, 3 * u + 1)],
                [(256, 1600, 16 * u + 17)], [(512, 1600, 18 * u + u // 2 + 1)], [(70, 1552, 22 * u)]]
    if dtype_name == "fp8":
        launches.append([(257, 16, 8 * u + 5)])
    for shapes in launches:
        tiles = sum(-(-M // 256) * -(-N // u) for M, K, N in shapes)
        assert tiles > W_ and 0 < tiles % W_ <= 3 * W_ // 8
        keep, outs, want = [], [], []
        def stage(M, K, N):
            X = rng.integers(-2, 3, (M, K)).astype(np.float32)
            Ws = [rng.integers(-1, 2, (K, N)).astype(np.float32) for _ in range(2 if gated else 1)]
            b = None if gated else rng.integers(-8, 9, N).astype(np.float32)
            dX = R.device_tensor_from_bits(U.to_bits(X, dtype_name), dt, U.DEV)
            dW = [R.pack_weights(R.device_tensor_from_bits(U.to_bits(w, dtype_name), dt, U.DEV), dt) for w in Ws]
            db = None if b is None else torch.from_numpy(b).to(U.DEV)
            dY = torch.zeros((M, N), dtype=torch.bfloat16, device=U.DEV)
            keep.extend([dX, db] + dW)
            outs.append(dY)
            if gated:
                z, up = X.astype(np.float64) @ Ws[0], X.astype(np.float64) @ Ws[1]
                want.append(z / (1 + np.exp(-z)) * up)
                return R.group_args(dX, dW[0], dY, M, K, N, "swiglu", W2=dW[1])
            want.append(ref.dense_forward(X.astype(np.float64), Ws[0].astype(np.float64), b, "relu"))
            return R.group_args(dX, dW[0], dY, M, K, N, "relu", bias=db)
        args = [stage(*sh) for sh in shapes]
        other = stage(65, shapes[0][1] + 64, 40)
        bits = []
        for groups in (args, args + [other]):
            plan = R.LaunchPlan(np.array(groups, dtype=B.GROUP_ARGS), dt, U.DEV, W_)
            assert int(plan.classes[-1][1]) == 256 and plan.n_panel_split_tiles == 0
            for rep in range(2):
                for y in outs:
                    y.fill_(float("nan"))
                R.grouped_forward(plan, B.EPARA_BF16)
                torch.cuda.synchronize()
            bits.append([y.view(torch.int16).clone() for y in outs[:len(shapes)]])
        for sh, quarters, whole, y, w in zip(shapes, *bits, outs, want):
            assert torch.equal(quarters, whole), sh
            if gated:
                assert_close(U.fetch(y), w, TOL[dtype_name], str(sh))
            else:
                assert np.array_equal(U.fetch(y), ref.bf16_decode(ref.bf16_encode(w))), sh


# ---- weights read with the non-temporal hint ----------------------------------------------------

@pytest.mark.parametrize("dtype_name,gated", [("bf16", False), ("bf16", True), ("fp8", False), ("fp8", True)])
def test_launches_too_large_for_the_last_level_cache_give_the_bits_of_their_groups_alone(dtype_name, gated):
    """Launches of more than 112 MB of weights (gated 192) read those of streaming tiles and of block tiles of a single row tile with another kernel
    than smaller ones: one batch of each streaming class, block tiles of 65 and 128 rows and two row tiles; sums of small integers: the bits of
    the same groups launched one by one, which stay below the line, and the oracle's."""
    rng = np.random.default_rng(37)
    dt, esz, K = B.DTYPE_BY_NAME[dtype_name], 2 if dtype_name == "bf16" else 1, 4096
    columns = -(-(200 if gated else 120) * 10 ** 6 // ((2 if gated else 1) * esz * K)) // 6
    shapes = [(M, K, columns + d) for d, M in enumerate((5, 20, 50, 65, 128, 129, 7))]
    keep, outs, want, args = [], [], [], []
    for M, _, N in shapes:
        X = rng.integers(-2, 3, (M, K)).astype(np.float32)
        Ws = [rng.integers(-1, 2, (K, N), dtype=np.int8).astype(np.float32) for _ in range(2 if gated else 1)]
        dX = R.device_tensor_from_bits(U.to_bits(X, dtype_name), dt, U.DEV)
        dW = [R.pack_weights(R.device_tensor_from_bits(U.to_bits(w, dtype_name), dt, U.DEV), dt) for w in Ws]
        dY = torch.zeros((M, N), dtype=torch.bfloat16, device=U.DEV)
        keep.extend([dX] + dW)
        outs.append(dY)
        z = [X.astype(np.float64) @ w for w in Ws]
        want.append(z[0] / (1 + np.exp(-z[0])) * z[1] if gated else np.maximum(z[0], 0))
        args.append(R.group_args(dX, dW[0], dY, M, K, N, "swiglu" if gated else "relu", W2=dW[1] if gated else None))
    assert sum(K * N * esz * (2 if gated else 1) for _, K, N in shapes) > (192e6 if gated else 112e6)
    bits = []
    for launches in ([args], [[a] for a in args]):
        for y in outs:
            y.fill_(float("nan"))
        for groups in launches:
            plan = R.LaunchPlan(np.array(groups, dtype=B.GROUP_ARGS), dt, U.DEV)
            assert len(groups) == 1 or int(plan.classes[-1][1]) == 128
            R.grouped_forward(plan, B.EPARA_BF16)
            torch.cuda.synchronize()
        bits.append([y.view(torch.int16).clone() for y in outs])
    for sh, together, alone, y, w in zip(shapes, *bits, outs, want):
        assert torch.equal(together, alone), sh
        if gated:
            assert_close(U.fetch(y), w, TOL[dtype_name], str(sh))
        else:
            assert np.array_equal(U.fetch(y), ref.bf16_decode(ref.bf16_encode(w))), sh


@pytest.mark.parametrize("K", [16, 136, 392, 1040])
def test_block_tiles_of_a_short_last_row_tile_give_the_bits_of_panel_tiles(K):
    """Gated bf16 block tiles, one row to 33 rows past one, two and three row tiles, next to groups without such a tile; ragged
    columns, K of one pair of stages, of both phases of the ring and ragged.  Sums of small integers: the bits of panel tiles, within the tolerance of the oracle."""
    rng = np.random.default_rng(43)
    rows, N = (129, 159, 160, 161, 256, 257, 288, 289, 385, 70, 128), 136
    keep, outs, want, args = [], [], [], []
    for M in rows:
        X = rng.integers(-2, 3, (M, K)).astype(np.float32)
        Ws = [rng.integers(-1, 2, (K, N)).astype(np.float32) for _ in range(2)]
        dX = R.device_tensor_from_bits(casts.bf16_bits(X), B.EPARA_BF16, U.DEV)
        dW = [R.pack_weights(R.device_tensor_from_bits(casts.bf16_bits(w), B.EPARA_BF16, U.DEV), B.EPARA_BF16) for w in Ws]
        dY = torch.zeros((M, N), dtype=torch.bfloat16, device=U.DEV)
        keep.extend([dX] + dW)
        outs.append(dY)
        z, u = X.astype(np.float64) @ Ws[0], X.astype(np.float64) @ Ws[1]
        want.append(z / (1 + np.exp(-z)) * u)
        args.append(R.group_args(dX, dW[0], dY, M, K, N, "swiglu", W2=dW[1]))
    bits = []
    for n_workgroups, tall in ((256, 128), (64, 256)):
        plan = R.LaunchPlan(np.array(args, dtype=B.GROUP_ARGS), B.EPARA_BF16, U.DEV, n_workgroups)
        assert int(plan.classes[-1][1]) == tall
        for rep in range(2):
            for y in outs:
                y.fill_(float("nan"))
            R.grouped_forward(plan, B.EPARA_BF16)
            torch.cuda.synchronize()
        bits.append([y.view(torch.int16).clone() for y in outs])
    for M, block, panel, y, w in zip(rows, *bits, outs, want):
        assert torch.equal(block, panel), M
        assert_close(U.fetch(y), w, TOL["bf16"], str(M))


@pytest.mark.parametrize("dtype_name,gated", [("bf16", True), ("bf16", False), ("fp8", True)])
def test_launches_of_some_of_the_tiles_write_those_and_nothing_else(dtype_name, gated):
    """A service's rows in two launches: the last row tiles in one, the others in another.  Each writes its own rows, with the bits of a launch of all
    tiles.  Last row tiles of one row, up to 32 and more, behind one whole row tile and two."""
    rng = np.random.default_rng(47)
    dt, rows, K, N, W_ = B.DTYPE_BY_NAME[dtype_name], (129, 130, 160, 161, 258, 288), 264 if dtype_name == "bf16" else 272, 136, 256
    keep, outs, args = [], [], []
    for M in rows:
        X = rng.integers(-2, 3, (M, K)).astype(np.float32)
        dX = R.device_tensor_from_bits(U.to_bits(X, dtype_name), dt, U.DEV)
        dW = [R.pack_weights(R.device_tensor_from_bits(U.to_bits(rng.integers(-1, 2, (K, N)).astype(np.float32), dtype_name), dt, U.DEV), dt) for _ in range(2 if gated else 1)]
        outs.append(torch.zeros((M, N), dtype=torch.bfloat16, device=U.DEV))
        keep.extend([dX] + dW)
        args.append(R.group_args(dX, dW[0], outs[-1], M, K, N, "swiglu" if gated else "relu", W2=dW[1] if gated else None))
    plan = R.LaunchPlan(np.array(args, dtype=B.GROUP_ARGS), dt, U.DEV, W_)
    assert int(plan.classes[-1][1]) == 128 and plan.n_panel_split_tiles == 0
    R.grouped_forward(plan, B.EPARA_BF16)
    torch.cuda.synchronize()
    whole = [y.view(torch.int16).clone() for y in outs]
    last = np.array([t["m0"] + t["rows"] == rows[t["group"]] for t in plan.tiles])
    for chosen in (last, ~last):
        tiles = np.ascontiguousarray(plan.tiles[chosen])
        order = np.full(-(-len(tiles) // W_) * W_, -1, dtype=np.int32)
        order[: len(tiles)] = np.arange(len(tiles))
        d_tiles, d_order = R._upload_all([tiles, order], U.DEV)
        launch = B.Launch(B._ptr(plan.args), plan.d_args.data_ptr(), B._ptr(tiles), d_tiles.data_ptr(), d_order.data_ptr(), len(tiles), len(order), W_, len(rows), None, 0, 0, 0)
        for y in outs:
            y.fill_(float("nan"))
        empty = outs[0].view(torch.int16)[0, 0].item()
        B.epara_grouped_forward(launch, dt, B.EPARA_BF16, R.current_stream_handle())
        torch.cuda.synchronize()
        for M, y, w in zip(rows, outs, whole):
            first = (M - 1) // 128 * 128
            got, mine = y.view(torch.int16), slice(first, M) if chosen is last else slice(0, first)
            other = slice(0, first) if chosen is last else slice(first, M)
            assert torch.equal(got[mine], w[mine]) and bool((got[other] == empty).all()), (M, chosen is last)


@pytest.mark.parametrize("dtype_name,gated", [("bf16", True), ("fp8", True), ("fp8", False)])
def test_entries_that_name_a_part_are_whole_tiles_where_nothing_is_visited_in_parts(dtype_name, gated):
    """Panel tiles of gated bf16 and fp8 launches are never visited in parts of K: an order whose entries name parts all the same gives the bits of the
    planner's, in whole rounds and in a last one that is cut into quarters."""
    rng = np.random.default_rng(53)
    dt, u, W_, K, M = B.DTYPE_BY_NAME[dtype_name], 128 if gated else 256, 16, 1552, 257
    N = 9 * u - 5                                                # 18 tiles
    X = rng.integers(-2, 3, (M, K)).astype(np.float32)
    dX = R.device_tensor_from_bits(U.to_bits(X, dtype_name), dt, U.DEV)
    dW = [R.pack_weights(R.device_tensor_from_bits(U.to_bits(rng.integers(-1, 2, (K, N)).astype(np.float32), dtype_name), dt, U.DEV), dt) for _ in range(2 if gated else 1)]
    dY = torch.zeros((M, N), dtype=torch.bfloat16, device=U.DEV)
    plan = R.LaunchPlan(np.array([R.group_args(dX, dW[0], dY, M, K, N, "swiglu" if gated else "relu", W2=dW[1] if gated else None)], dtype=B.GROUP_ARGS), dt, U.DEV, W_)
    assert len(plan.tiles) == 18 and int(plan.classes[-1][1]) == 256 and plan.n_panel_split_tiles == 0
    bits = []
    for part, parts in ((0, 1), (0, 2), (1, 2), (2, 4)):
        order = np.where(plan.order < 0, plan.order, plan.order | part << 24 | (parts - 1) << 28).astype(np.int32)
        d_order, = R._upload_all([order], U.DEV)
        launch = B.Launch(B._ptr(plan.args), plan.d_args.data_ptr(), B._ptr(plan.tiles), plan.d_tiles.data_ptr(), d_order.data_ptr(), len(plan.tiles), len(order), W_, 1, None, 0, 0, 0)
        dY.fill_(float("nan"))
        B.epara_grouped_forward(launch, dt, B.EPARA_BF16, R.current_stream_handle())
        torch.cuda.synchronize()
        bits.append(dY.view(torch.int16).clone())
    assert not torch.isnan(bits[0].view(torch.bfloat16)).any() and all(torch.equal(b, bits[0]) for b in bits[1:])


@pytest.mark.parametrize("dtype_name,gated,out_name", [("bf16", True, "bf16"), ("fp8", True, "bf16"), ("fp8", True, "fp8"), ("fp8", False, "bf16")])
def test_last_rounds_in_quarters_on_whole_grids(dtype_name, gated, out_name):
    """The same comparison on grids of 128 and 256 workgroups, cut into panel tiles whatever a plan would choose: 8 to 96 tiles past one and two whole rounds,
    spread over two and four words of 64 slots, several of them per group of workgroups of a die; E4M3 outputs too.  Nothing may stay unwritten."""
    gen = torch.Generator(device=U.DEV)
    gen.manual_seed(59)
    dt, out_dt, u = B.DTYPE_BY_NAME[dtype_name], B.DTYPE_BY_NAME[out_name], 128 if gated else 256
    K = 1552 if dtype_name == "bf16" else 16
    stored = lambda x: x.to(torch.bfloat16) if dt == B.EPARA_BF16 else x.to(torch.float8_e4m3fn).view(torch.uint8)
    ints = lambda lo, hi, shape: torch.randint(lo, hi + 1, shape, generator=gen, device=U.DEV).float()
    launches = [(256, [(700, 88 * u)]), (256, [(1000, 72 * u - 3)]), (256, [(970, 88 * u - 9)]), (256, [(600, 100 * u + 1), (70, 49 * u)]), (256, [(1030, 109 * u)]),
                (128, [(1000, 34 * u - 5)]), (128, [(300, 83 * u)]), (128, [(257, 144 * u - 1)])]
    rests = []
    for W_, shapes in launches:
        args, outs, wants, keep = [], [], [], []
        for M, N in shapes + [(65, 40)]:
            k = K if len(args) < len(shapes) else K + 64
            X, Ws = ints(-2, 2, (M, k)), [ints(-1, 1, (k, N)) for _ in range(2 if gated else 1)]
            dX, dW = stored(X), [R.pack_weights(stored(w), dt) for w in Ws]
            dY = torch.empty((M, N), dtype=R.TORCH_DTYPE[out_dt], device=U.DEV)
            keep.extend([dX] + dW)
            outs.append(dY)
            z = [X.double() @ w.double() for w in Ws]
            wants.append(z[0] / (1 + torch.exp(-z[0])) * z[1] if gated else z[0].clamp(min=0))
            args.append(R.group_args(dX, dW[0], dY, M, k, N, "swiglu" if gated else "relu", W2=dW[1] if gated else None))
        bits = []
        for n in (len(shapes), len(shapes) + 1):                 # with the group of another K: whole tiles
            table = np.array(args[:n], dtype=B.GROUP_ARGS)
            groups = R._group_desc(table)
            cls, n_stream = B.epara_kernel_classes(dt, int(gated), 0)
            tiles = B.epara_plan_groups(groups, cls)[3]
            order = B.epara_schedule_tiles(groups, cls, n_stream, tiles, W_, 8, 1, 4)
            if n == len(shapes):
                rests.append((len(tiles) // W_, len(tiles) % W_))
                assert rests[-1][0] >= 1 and 0 < 8 * rests[-1][1] <= 3 * W_, (W_, shapes, rests[-1])
            d = R._upload_all([table, tiles, order], U.DEV)
            launch = B.Launch(B._ptr(table), d[0].data_ptr(), B._ptr(tiles), d[1].data_ptr(), d[2].data_ptr(), len(tiles), len(order), W_, n, None, 0, 0, 0)
            for y in outs:
                y.view(torch.uint8).fill_(0xFF)                  # a NaN in either type
            B.epara_grouped_forward(launch, dt, out_dt, R.current_stream_handle())
            torch.cuda.synchronize()
            bits.append([y.view(torch.uint8).clone() for y in outs[:len(shapes)]])
        for (M, N), quarters, whole, y, want in zip(shapes, *bits, outs, wants):
            assert torch.equal(quarters, whole), (W_, M, N)
            if out_dt == B.EPARA_FP8_E4M3:
                assert not bool((quarters == 0xFF).any()), (W_, M, N)
            elif gated:
                assert_close(U.fetch(y), want.cpu().numpy(), TOL[dtype_name], str((W_, M, N)))
            else:
                assert torch.equal(y, want.to(torch.bfloat16)), (W_, M, N)
    assert {r for r, _ in rests} == {1, 2} and min(r for _, r in rests) == 8 and max(r for _, r in rests) == 96, rests
