"""GPU parity: the HIP path (through the C boundary) against the float64 CPU oracle, element by element.

Tolerances (tests/harness.py): parameters <= 1e-4, accumulators <= 1e-5 in the metric
max_i |a_i - b_i| / (|b_i| + rms(b)) per tensor; both sides use the same float32 inputs and scalars.
"""
import numpy as np
import pytest

import workloads as W
from tests import harness as Hn
from tests.planner import plan
from tests.test_planner_cpu import NARROW, UNALIGNED

pytestmark = pytest.mark.gpu


def _specs(shapes):
    return [W.TensorSpec(f"t{i}", tuple(s)) for i, s in enumerate(shapes)]


def test_config1_small_fc_free_running():
    wl = W.get_workload(1)
    cfg = Hn.make_cfg("small_fc_lopt")
    w = W.small_fc_weights(0, 32)
    worst = Hn.run_free(Hn.Case(1, wl.tensors, wl.grad_kind), cfg, w, wl.steps, verbose=True)
    print("config1 worst:", worst)


ODD_SHAPES = [(7, 13), (5,), (1,), (3, 1), (300, 257), (65, 1000), (2, 3, 5), (1, 1, 33), (130, 260), (1030,)]


@pytest.mark.parametrize("hidden", [3, 5, 12, 32])
def test_small_fc_odd_shapes_and_hidden_widths(hidden):
    cfg = Hn.make_cfg("small_fc_lopt", hidden=hidden)
    w = Hn.random_weights(cfg, seed=hidden)
    Hn.run_free(Hn.Case(101, _specs(ODD_SHAPES)), cfg, w, 4, lr_fn=lambda t: 0.5, wd=0.01)


@pytest.mark.parametrize("hidden,lstm_hidden,n_bank", [(4, 16, 8), (2, 33, 5), (4, 512, 256), (7, 64, 16)])
def test_velo_odd_shapes(hidden, lstm_hidden, n_bank):
    cfg = Hn.make_cfg("velo", hidden=hidden, lstm_hidden=lstm_hidden, n_bank=n_bank)
    w = Hn.random_weights(cfg, seed=3)
    Hn.run_free(Hn.Case(102, _specs(ODD_SHAPES), "gauss_logscale"), cfg, w, 4, lr_fn=lambda t: 0.5, wd=0.01)


@pytest.mark.parametrize("kind", ["small_fc_lopt", "velo"])
def test_unaligned_rows_at_every_sweep_boundary(kind):
    # rows that are not 16-byte aligned (n % 4 != 0) take the statistics pass one column per lane, 64 columns per sweep,
    # four sweeps per 256-column tile: widths just below and above every sweep and tile boundary, heights below, at and
    # above a tile's 64 rows (the apply kernels see the same widths through their ragged last strips)
    cfg = Hn.make_cfg(kind) if kind == "small_fc_lopt" else Hn.make_cfg(kind, lstm_hidden=32, n_bank=8)
    w = Hn.random_weights(cfg, seed=21)
    shapes = [(9, 63), (70, 65), (64, 127), (3, 129), (130, 191), (65, 193), (11, 255), (66, 257), (5, 321), (2, 513)]
    worst = Hn.run_free(Hn.Case(112, _specs(shapes), "gauss_logscale"), cfg, w, 3, lr_fn=lambda t: 0.5, wd=0.01)
    assert worst["param"] <= Hn.TOL_PARAM


@pytest.mark.parametrize("state_pass", ["apply", "stats"])
def test_velo_one_column_per_lane_path_at_segment_and_row_boundaries(state_pass):
    # the width-4 kernel on rows that are not 16-byte aligned: one column per lane, four rows per trip, wavefronts on 64-column
    # segments that share out the rows of narrow tiles: one, two, three and four segments, heights around the trip of four rows
    # and the tile (eight rows on a list this short); beside them 16-byte aligned rows off and on the 128-byte grid
    cfg = Hn.make_cfg("velo", lstm_hidden=32, n_bank=8, state_pass=state_pass)
    w = Hn.random_weights(cfg, seed=22)
    shapes = [(1, 1), (2, 3), (17, 61), (15, 65), (33, 129), (64, 190), (65, 257), (130, 318), (257, 1), (4, 449), (67, 260), (66, 288)]
    worst = Hn.run_free(Hn.Case(113, _specs(shapes), "gauss_logscale"), cfg, w, 3, lr_fn=lambda t: 0.5, wd=0.01)
    assert worst["param"] <= Hn.TOL_PARAM


@pytest.mark.parametrize("state_pass", ["apply", "stats"])
def test_strip_tiles_of_every_number_of_row_pairs(state_pass):
    # apply tiles of 16 rows (487 of them) and last tiles of 1 to 16 rows: one to eight pairs through the pipeline, odd and even
    # numbers of its two-pair turns, a last pair of one row
    cfg = Hn.make_cfg("small_fc_lopt", state_pass=state_pass)
    w = Hn.random_weights(cfg, seed=25)
    shapes = [(16 + r, 100 + r) for r in range(16)] + [(900, 1000)]
    assert max(h for h, _ in plan(shapes)["atile_runs"]) == 16
    worst = Hn.run_free(Hn.Case(125, _specs(shapes), "gauss_logscale"), cfg, w, 2, lr_fn=lambda t: 0.5, wd=0.01)
    assert worst["param"] <= Hn.TOL_PARAM


@pytest.mark.parametrize("hidden", [32, 19])
@pytest.mark.parametrize("shapes", [[(300, 300), (7, 130), (1, 40)], [(100, 300)] * 44])
def test_strip_workgroups_that_form_their_tensors_scales(shapes, hidden):
    # up to one round of 512 apply tiles the strip kernel forms the scales and the first layer from the partials itself; the second
    # list has more and takes the launch in between. Also a width that is padded to 32; s_f as the workspace holds it is compared too.
    # Tensors of at most 90 000 elements; a million has a test of its own below.
    cfg = Hn.make_cfg("small_fc_lopt", hidden=hidden)
    w = Hn.random_weights(cfg, seed=28)
    form = plan(shapes, hidden=hidden)
    assert form["short_list"] == 1 and form["fold_finalize"] == (form["n_atiles"] <= 512) == (len(shapes) == 3)
    worst = Hn.run_free(Hn.Case(128, _specs(shapes), "gauss_logscale"), cfg, w, 2, lr_fn=lambda t: 0.5, wd=0.01)
    assert worst["param"] <= Hn.TOL_PARAM


@pytest.mark.parametrize("weights_seed", [27, 28])
def test_strip_workgroups_form_the_scales_of_a_million_elements_as_k_finalize_does(weights_seed):
    # The same tensor alone (its workgroups form the scales) and in a list of more than one round of apply tiles (a launch in between
    # does): the same bits, s_f included. Against the oracle the bar of 1e-4 on the update does not hold for every such tensor: in the
    # first steps 1 / sqrt(V) of an element of small gradient is a feature of up to sqrt(N), and the fp16 pairs round its products by
    # 2^-22 each way. That adds at most 2^-21 sqrt(N) of the rms update, 4.8e-4 here (weights of seed 27: 1.008e-4 in all).
    import torch
    import paper_2506_10315_amd as P
    cfg = Hn.make_cfg("small_fc_lopt")
    w = Hn.random_weights(cfg, seed=weights_seed)
    case = Hn.Case(128, _specs([(1000, 1000)]), "gauss_logscale")
    outs = []
    for rest in ([], [(100, 300)] * 44):
        shapes = [(1000, 1000)] + rest
        form = plan(shapes)
        assert (form["short_list"], form["fold_finalize"], form["tensors"][0]["TR"]) == (1, not rest, 8)
        opt = P.LearnedOptimizer(cfg, w, shapes)
        p = [torch.from_numpy(case.p0(0)).to("cuda:0")] + [torch.zeros(s, device="cuda:0") for s in rest]
        for t in range(2):
            g = [torch.from_numpy(case.grad(0, t)).to("cuda:0")] + [torch.ones(s, device="cuda:0") for s in rest]
            opt.step(p, g, lr=0.5, weight_decay=0.01, step=t)
        outs.append(torch.cat([p[0].reshape(-1), opt.state[0], opt.stats()[0]]).view(torch.int32).cpu())
        opt.close()
    assert torch.equal(*outs)
    worst = Hn.run_free(case, cfg, w, 2, lr_fn=lambda t: 0.5, wd=0.01, tol_delta=Hn.TOL_DELTA + 2.0 ** -21 * 1000)
    assert worst["param"] <= Hn.TOL_PARAM


@pytest.mark.parametrize("rows", [6144, 6145])
@pytest.mark.parametrize("kind,state_pass", [("small_fc_lopt", "apply"), ("small_fc_lopt", "stats"), ("velo", "apply")])
def test_row_and_column_means_at_the_limit_of_a_short_list(kind, state_pass, rows):
    # up to 96 tiles of 64 rows the statistics workgroups finish the row and column means themselves; one row more and a launch of
    # its own does. 96 column tiles; rows and columns at the edges of a tile of the sums and of the statistics
    cfg = Hn.make_cfg(kind, state_pass=state_pass) if kind == "small_fc_lopt" else Hn.make_cfg(kind, lstm_hidden=33, n_bank=8,
                                                                                             state_pass=state_pass)
    w = Hn.random_weights(cfg, seed=26)
    shapes = [(rows, 5), (3, 24576), (64, 256), (65, 257), (63, 255), (129, 1100), (1, 1), (1, 300)]
    assert (plan(shapes, kind=kind)["n_rcitems"] == 0) == (rows == 6144)
    worst = Hn.run_free(Hn.Case(126, _specs(shapes), "gauss_logscale"), cfg, w, 3, lr_fn=lambda t: 0.5, wd=0.01)
    assert worst["param"] <= Hn.TOL_PARAM


@pytest.mark.parametrize("cols", [20000, 19999])
@pytest.mark.parametrize("rows", [64, 100, 128, 256, 1025])
def test_column_means_of_short_lists_lose_no_bits_in_their_partial_sums(rows, cols):
    # With beta_5..7 = 0 the state's c_k are the column means themselves, rounded once to fp32. Before that only the sums of up to
    # eight squares in a lane are formed in fp32, at least 8 ceil(rows / 64) of them of about equal size: the k-th of eight roundings,
    # of rms 2^-24 / sqrt(3) at most, hits k / 8 of a sum, 1.79 together, and 1.2 allows for the sums' spread. fp32 sums over the
    # lanes and fp32 partials were 3.2e-8 to 4.3e-8 off here, 2.8e-8 is what the final rounding and the lanes' sums give.
    import torch
    import paper_2506_10315_amd as P
    shapes = [(rows, cols)]
    assert plan(shapes, hidden=4)["short_list"] == 1
    cfg = Hn.make_cfg("small_fc_lopt", hidden=4)
    cfg.fac_decay[:] = [0.0] * 3
    opt = P.LearnedOptimizer(cfg, Hn.random_weights(cfg, seed=5), shapes)
    gen = torch.Generator(device="cuda:0").manual_seed(rows)
    g = torch.randn(rows, cols, device="cuda:0", generator=gen) * 1e-3
    p = torch.zeros(rows, cols, device="cuda:0")
    opt.step([p], [g], lr=0.0)
    exact = g.double().square().mean(0)
    rms = lambda x: float(((x.double() - exact) / exact).square().mean().sqrt())
    bound = (rms(exact.float()) ** 2 + (1.2 * 1.79 * 2.0 ** -24 / 3 ** 0.5) ** 2 / (8 * -(-rows // 64))) ** 0.5
    for c in opt.state_views(0)["c"]:
        assert rms(c.reshape(-1)) <= bound
    opt.close()


@pytest.mark.parametrize("tall", [[], [(6145, 3)]])
@pytest.mark.parametrize("kind,state_pass", [("small_fc_lopt", "apply"), ("velo", "apply"), ("velo", "stats")])
def test_rows_of_a_multiple_of_4_kb(kind, state_pass, tall):
    # widths that are a multiple of 1024 are walked by groups of four tiles (up to 3072 columns) or from a start that differs
    # from tile to tile (beyond): heights below, at and above a tile and its quarters; 1280 columns keep the plain walk. In the
    # VeLO apply pass of any list; in the statistics pass of lists that are not short, which a tall tensor makes of this one
    cfg = Hn.make_cfg(kind, state_pass=state_pass) if kind == "small_fc_lopt" else Hn.make_cfg(kind, lstm_hidden=32, n_bank=8,
                                                                                             state_pass=state_pass)
    w = Hn.random_weights(cfg, seed=24)
    shapes = [(70, 1024), (1, 1024), (9, 2048), (64, 2048), (131, 3072), (3, 3072), (67, 4096), (2, 5120), (150, 4096), (66, 1280)] + tall
    assert plan(shapes, kind=kind, lstm_hidden=32, n_bank=8)["short_list"] == (not tall)
    worst = Hn.run_free(Hn.Case(115, _specs(shapes), "gauss_logscale"), cfg, w, 2, lr_fn=lambda t: 0.5, wd=0.01)
    assert worst["param"] <= Hn.TOL_PARAM


@pytest.mark.parametrize("hidden,lstm_hidden,n_bank,count", [(3, 37, 64, 7), (7, 64, 128, 33), (4, 5, 300, 3), (8, 200, 400, 40),
                                                             (3, 37, 64, 97), (7, 64, 128, 99), (4, 5, 300, 97), (8, 200, 400, 97), (2, 130, 64, 128),
                                                             (7, 64, 128, 1030)])
def test_velo_folded_head_and_lstm_octets(hidden, lstm_hidden, n_bank, count):
    # banks large enough for the head's two products to be folded into one matrix: padded widths, more than 256 columns (the
    # step-size column in a second block), LSTM widths off the octet and unit grids, tensor counts around a block of 32, and
    # the batched form. Up to 96 tensors in column blocks with the recurrent product ahead, then one workgroup per tensor behind
    # the whole LSTM. Tensors have at least 8 elements: the statistic of M_i / sqrt(V) of a single element carries the
    # relative rounding error of beta M + (1 - beta) g, 2^-24 (|beta M| + |(1 - beta) g|) / |their sum|, which has no bound
    # when the two nearly cancel (a one-element tensor of this seed: factor 1005, 2.4e-5); in a mean over 8 the other terms
    # keep the sum's size.
    cfg = Hn.make_cfg("velo", hidden=hidden, lstm_hidden=lstm_hidden, n_bank=n_bank)
    w = Hn.random_weights(cfg, seed=40 + lstm_hidden)
    r = np.random.default_rng(78)
    shapes = [(7, 13), (33, 20)] + [(int(r.integers(8, 60)),) for _ in range(count - 2)]
    assert plan(shapes, kind="velo", hidden=hidden, lstm_hidden=lstm_hidden, n_bank=n_bank)["lstm_ahead"] == (count <= 96)
    worst = Hn.run_free(Hn.Case(116, _specs(shapes), "gauss_logscale"), cfg, w, 3, lr_fn=lambda t: 0.5, wd=0.01)
    assert worst["param"] <= Hn.TOL_PARAM


@pytest.mark.parametrize("hidden,lstm_hidden,n_bank,count", [(4, 1024, 256, 5), (4, 520, 300, 17), (5, 130, 200, 96), (5, 130, 200, 97),
                                                             (4, 9, 64, 16)])
def test_velo_recurrent_product_ahead_and_head_in_column_blocks(hidden, lstm_hidden, n_bank, count):
    # up to 96 tensors the LSTM's recurrent product is formed beside the row/column sums, in blocks of 16 tensors, and the head in
    # blocks of 32 columns; 97 tensors take one launch for each. Widths on and off the octet, one and two batches of head rows.
    # Two lists in one: tensor shapes below and above the limit of a short list (6145 rows), whose sums are another kernel
    cfg = Hn.make_cfg("velo", hidden=hidden, lstm_hidden=lstm_hidden, n_bank=n_bank)
    w = Hn.random_weights(cfg, seed=60 + lstm_hidden)
    r = np.random.default_rng(79)
    for first in ((7, 13), (6145, 3)):
        shapes = [first, (33, 20)] + [(int(r.integers(8, 60)),) for _ in range(count - 2)]
        form = plan(shapes, kind="velo", hidden=hidden, lstm_hidden=lstm_hidden, n_bank=n_bank)
        assert (form["short_list"], form["lstm_ahead"]) == (first == (7, 13), count <= 96)
        worst = Hn.run_free(Hn.Case(127, _specs(shapes), "gauss_logscale"), cfg, w, 3, lr_fn=lambda t: 0.5, wd=0.01)
        assert worst["param"] <= Hn.TOL_PARAM


@pytest.mark.parametrize("count", [1, 2, 3, 5, 8, 9])
def test_velo_lstm_launch_that_forms_its_inputs(count):
    # up to eight tensors share the LSTM launch's eight half wavefronts, eight, four, two or one to a tensor; nine take the launch in
    # between. Second list: 63 and 65 statistics tiles in the largest tensor, one and two batches of a half wavefront (or, for a few
    # tensors, one of several), and one tile more than two batches of one
    cfg = Hn.make_cfg("velo", lstm_hidden=40, n_bank=64)
    w = Hn.random_weights(cfg, seed=80 + count)
    small = [(7, 13), (33, 20), (300,), (64, 256), (9, 300), (17, 17), (1, 40), (80, 3), (5, 60)]
    for big in ((64, 256), (8 * 63, 40), (8 * 65, 40)):
        form = plan([big] + small[:count - 1], kind="velo", lstm_hidden=40, n_bank=64)
        assert form["lstm_ahead"] == 1 and form["fold_finalize"] == (count <= 8 and (count <= 4 or big != (8 * 65, 40)))
        worst = Hn.run_free(Hn.Case(129, _specs([big] + small[:count - 1]), "gauss_logscale"), cfg, w, 3, lr_fn=lambda t: 0.5, wd=0.01)
        assert worst["param"] <= Hn.TOL_PARAM


def _velo_weight_views(w, cfg):
    """The sections of a VeLO weight blob (include/lopt.h) as views of `w`."""
    HL, K, h = int(cfg.lstm_hidden), int(cfg.n_bank), int(cfg.hidden)
    P_ = 29 * h + h + h * h + h + 2 * h + 2
    out, o = {}, 0
    for name, shape in (("Wx", (48, 4, HL)), ("Wh", (HL, 4, HL)), ("Wg", (HL, 4, HL)), ("b", (4, HL)), ("Wa", (HL, K)), ("ba", (K,)),
                        ("ws", (HL,)), ("bs", (1,)), ("B", (K, P_))):
        n = int(np.prod(shape))
        out[name] = w[o:o + n].reshape(shape)
        o += n
    assert o == w.size
    return out


@pytest.mark.parametrize("count", [3, 1030])
def test_velo_bank_products_beyond_the_fp32_range(count):
    # finite weights whose product W_a B is not: a unit whose output is exactly 0 (its candidate gate has no weights) with
    # coefficients of 1e30 beside a bank of 1e10; h W_a and (h W_a) B stay of ordinary size
    cfg = Hn.make_cfg("velo", lstm_hidden=64, n_bank=128)
    w = Hn.random_weights(cfg, seed=50)
    v = _velo_weight_views(w, cfg)
    for name in ("Wx", "Wh", "Wg"):
        v[name][:, 2, 5] = 0.0
    v["b"][2, 5] = 0.0
    v["Wa"][:] *= 1e-10
    v["ba"][:] *= 1e-10
    v["B"][:] *= 1e10
    v["Wa"][5] = np.where(np.arange(128) % 3 == 0, -1e30, 1e30)
    r = np.random.default_rng(79)
    shapes = [(7, 13), (33, 20)] + [(int(r.integers(8, 60)),) for _ in range(count - 2)]
    worst = Hn.run_free(Hn.Case(117, _specs(shapes), "gauss_logscale"), cfg, w, 2, lr_fn=lambda t: 0.5, wd=0.01)
    assert worst["param"] <= Hn.TOL_PARAM


@pytest.mark.parametrize("count", [3, 1030])
def test_velo_step_size_is_summed_with_few_roundings(count):
    # ln(lambda) = h . ws over 512 equal terms of about 0.12, whose long serial sums round the same way again and again (the
    # chosen ws: 12 units of 2^-24 after 32 + 16 terms, 20 after 128 + 4; 0.4 from eight terms a lane and a tree, in any of
    # the three floats next to tanh(1)). One rounding for the products and up to three for eight terms a lane are admitted,
    # the tree is exact; 8 units for expf, the MLP's output layer and the update. W_a and B make the direction exactly 1.
    import torch
    import paper_2506_10315_amd as P
    cfg = Hn.make_cfg("velo")
    w = np.zeros(P.weights_count(cfg), np.float32)
    v = _velo_weight_views(w, cfg)
    v["b"][:] = 20.0                       # saturated gates: c = 1, h = tanh(1) in every unit
    v["ba"][0] = 1.0
    v["B"][0, -2] = 1.0                    # b3, direction
    v["ws"][:] = 0.15736201
    shapes = [(8, 16)] * count
    opt = P.LearnedOptimizer(cfg, w, shapes)
    p = [torch.zeros(s, device="cuda:0") for s in shapes]
    g = [torch.full(s, 1e-3, device="cuda:0") for s in shapes]
    opt.step(p, g, lr=1.0, step=0, loss=1.0)
    torch.cuda.synchronize()
    for i in (0, count - 1):
        h = opt.state_views(i)["h"].cpu().numpy().astype(np.float64)
        ln = float(h @ v["ws"].astype(np.float64))
        assert 61.0 < ln < 62.0
        lam = -p[i].cpu().numpy().astype(np.float64) / float(np.float32(cfg.step_mult))
        assert np.max(np.abs(lam / np.exp(ln) - 1.0)) <= (4 * ln + 8) * 2.0 ** -24
    opt.close()


@pytest.mark.parametrize("lstm_hidden,count", [(100, 5), (512, 16), (1024, 96)])
def test_velo_step_size_of_short_lists_loses_no_bits_in_its_sum(lstm_hidden, count):
    # ln(lambda) = h . ws of some hundred terms of about one that cancel (ws orthogonal to every tensor's h, which does not depend on
    # it; 4 ws, so that fp32 products and sums are 5 to 20 units of 2^-24 off). In double only its own rounding is left, far below a
    # unit where it is near 0; 2 units for expf, 4 for the step size's way through the MLP's output layer and the update.
    import torch
    import paper_2506_10315_amd as P
    cfg = Hn.make_cfg("velo", lstm_hidden=lstm_hidden)
    w = Hn.random_weights(cfg, seed=70)
    v = _velo_weight_views(w, cfg)
    v["Wa"][:], v["ba"][:], v["B"][:], v["bs"][:] = 0.0, 0.0, 0.0, 0.0
    v["Wx"][:] *= 20.0                     # outputs of every size up to one, different for every tensor
    v["ba"][0] = 1.0
    v["B"][0, -2] = 1.0                    # b3, direction
    v["ws"][:] = 0.0
    shapes = [(8 + i, 16) for i in range(count)]
    gen = torch.Generator(device="cuda:0").manual_seed(3)
    g = [torch.randn(s, device="cuda:0", generator=gen) * 10.0 ** -(1 + i % 5) for i, s in enumerate(shapes)]

    def step():
        opt = P.LearnedOptimizer(cfg, w, shapes)
        p = [torch.zeros(s, device="cuda:0") for s in shapes]
        opt.step(p, g, lr=1.0, step=0, loss=1.0)
        h = np.stack([opt.state_views(i)["h"].cpu().numpy().astype(np.float64) for i in range(count)])
        opt.close()
        return h, [-x.cpu().numpy().astype(np.float64) / float(np.float32(cfg.step_mult)) for x in p]

    h, _ = step()
    r = np.random.default_rng(71).uniform(-4.0, 4.0, lstm_hidden)
    v["ws"][:] = r - h.T @ np.linalg.lstsq(h @ h.T, h @ r, rcond=None)[0]
    h2, lam = step()
    assert np.array_equal(h, h2)
    ln = h @ v["ws"].astype(np.float64)
    assert np.max(np.abs(ln)) < 1e-3 and np.max(np.abs(h * v["ws"]).sum(1)) > 0.2 * lstm_hidden
    assert max(np.max(np.abs(x / np.exp(l) - 1.0)) for x, l in zip(lam, ln)) <= 6 * 2.0 ** -24


@pytest.mark.parametrize("hidden,state_pass", [(1, "apply"), (4, "stats"), (8, "apply"), (9, "stats"), (16, "apply"), (16, "stats")])
def test_small_fc_narrow_widths_at_tile_boundaries(hidden, state_pass):
    # hidden widths up to 16 (padded to 4, 8, 16) run on fp32 matrix instructions over tiles of 128 columns, 64 columns a
    # wavefront: one segment, two segments, ragged second tiles, rows off and on the 16- and 128-byte grids, on tiles of the
    # least height (two rows at width 16, eight below); the accumulators written in either pass
    cfg = Hn.make_cfg("small_fc_lopt", hidden=hidden, state_pass=state_pass)
    w = Hn.random_weights(cfg, seed=30 + hidden)
    shapes = [(1, 1), (3, 15), (5, 17), (2, 63), (129, 64), (17, 65), (16, 127), (260, 128), (9, 129), (31, 193), (7, 256), (70, 300)]
    worst = Hn.run_free(Hn.Case(114, _specs(shapes), "gauss_logscale"), cfg, w, 3, lr_fn=lambda t: 0.5, wd=0.01)
    assert worst["param"] <= Hn.TOL_PARAM


@pytest.mark.parametrize("hidden", [4, 8, 16])
def test_small_fc_narrow_widths_on_full_tiles(hidden):
    # tiles of 128, 64 and 32 rows, one and two column segments, and more tiles than workgroups (tests/test_planner_cpu.py): the
    # row prefetch, the rows that wavefronts share and the tables of a workgroup's second tile
    cfg = Hn.make_cfg("small_fc_lopt", hidden=hidden)
    w = Hn.random_weights(cfg, seed=60 + hidden)
    worst = Hn.run_free(Hn.Case(118, _specs(NARROW), "gauss_logscale"), cfg, w, 2, lr_fn=lambda t: 0.5, wd=0.01)
    assert worst["param"] <= Hn.TOL_PARAM


@pytest.mark.parametrize("kind", ["small_fc_lopt", "velo"])
def test_unaligned_rows_on_tiles_of_ordinary_height(kind):
    # tiles of 64 and 320 rows whose wavefronts share one or two column segments and take several trips of four rows each, or
    # sit on three or four segments (tests/test_planner_cpu.py); small_fc_lopt for the statistics pass, which both share
    cfg = Hn.make_cfg(kind) if kind == "small_fc_lopt" else Hn.make_cfg(kind, lstm_hidden=32, n_bank=8)
    w = Hn.random_weights(cfg, seed=64)
    worst = Hn.run_free(Hn.Case(119, _specs(UNALIGNED), "gauss_logscale"), cfg, w, 2, lr_fn=lambda t: 0.5, wd=0.01)
    assert worst["param"] <= Hn.TOL_PARAM


@pytest.mark.parametrize("hidden,lstm_hidden,n_bank", [(3, 33, 5), (4, 512, 256)])
def test_velo_long_list_takes_the_batched_hypernetwork_head(hidden, lstm_hidden, n_bank):
    # from 1024 tensors on the head of the hypernetwork runs as two batched matrix products and a scatter kernel
    # instead of one workgroup per tensor: 1100 tensors (ragged last block of 32), odd and default widths
    cfg = Hn.make_cfg("velo", hidden=hidden, lstm_hidden=lstm_hidden, n_bank=n_bank)
    w = Hn.random_weights(cfg, seed=9)
    r = np.random.default_rng(77)
    shapes = [(int(r.integers(1, 40)),) for _ in range(1090)] + [(7, 13), (64, 256), (3, 1), (130, 260)] * 2 + [(33,), (5,)]
    assert len(shapes) == 1100
    worst = Hn.run_free(Hn.Case(109, _specs(shapes), "gauss_logscale"), cfg, w, 3, lr_fn=lambda t: 0.5, wd=0.01)
    assert worst["param"] <= Hn.TOL_PARAM


@pytest.mark.parametrize("state_pass", ["apply", "stats"])
def test_velo_config1_shapes_free_running_with_clip_active(state_pass):
    # gradients of order 0.1 so that the clipped-gradient feature differs from the gradient; the width-4 apply kernel
    # with the accumulator update in either pass
    cfg = Hn.make_cfg("velo", state_pass=state_pass)
    w = W.velo_weights(0)

    class BigGrad(Hn.Case):
        def grad(self, i, step):
            return (super().grad(i, step) * np.float32(100.0)).astype(np.float32)

    Hn.run_free(BigGrad(103, W.config1_shapes()), cfg, w, 6, lr_fn=lambda t: W.lr_at(W.get_workload(3), t), wd=0.01)


def test_tall_and_wide_tensors():
    # tall: more rows than 256 standard row tiles hold (the tile height grows); wide 1-D: many column tiles
    cfg = Hn.make_cfg("small_fc_lopt")
    w = W.small_fc_weights(1, 32)
    Hn.run_free(Hn.Case(104, _specs([(9000, 256), (5504,), (4100, 8), (40000, 4)]), "student_t3"), cfg, w, 3)


def _random_shapes(seed, count):
    """Seeded list of 1-D/2-D/3-D shapes with ragged sizes around the kernels' tile edges (4, 32, 64, 128, 256)."""
    r = np.random.default_rng(seed)
    edges = np.array([1, 2, 3, 4, 5, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257, 300, 513])
    shapes = []
    for _ in range(count):
        kind = r.integers(0, 10)
        a, b = int(r.choice(edges)), int(r.choice(edges))
        if r.integers(0, 2):
            a = int(r.integers(1, 400))
        if kind == 0:
            shapes.append((a,))
        elif kind == 1:
            shapes.append((int(r.integers(1, 4)), int(r.integers(1, 5)), b))
        else:
            shapes.append((a, b))
    return shapes


@pytest.mark.parametrize("kind,seed", [("small_fc_lopt", 11), ("small_fc_lopt", 12), ("velo", 13)])
def test_random_shape_lists(kind, seed):
    # shapes nobody picked by hand: every pass sees ragged first/last tiles in rows and columns
    cfg = Hn.make_cfg(kind) if kind == "small_fc_lopt" else Hn.make_cfg(kind, lstm_hidden=32, n_bank=8)
    w = Hn.random_weights(cfg, seed=seed)
    Hn.run_free(Hn.Case(110 + seed, _specs(_random_shapes(seed, 24)), "gauss_logscale"), cfg, w, 3,
                lr_fn=lambda t: 0.5, wd=0.01)


@pytest.mark.parametrize("variant,state_pass", [("valu", None), ("mfma_f32", None), ("mfma_f16s", "apply"),
                                                ("mfma_f16s", "stats")])
def test_every_apply_kernel_variant_matches_the_oracle(variant, state_pass):
    # the configuration's apply_kernel field selects the apply kernel for hidden width 32: vector ALU, fp32 MFMA, or
    # split-fp16 MFMA (the default), the last with the accumulator update in either pass. All must meet the same bar.
    cfg = Hn.make_cfg("small_fc_lopt", apply_kernel=variant, state_pass=state_pass)
    w = W.small_fc_weights(2, 32)
    shapes = [(256, 256), (256,), (64, 256), (300, 257), (33, 1000), (7,)]
    worst = Hn.run_free(Hn.Case(105, _specs(shapes), "student_t3"), cfg, w, 6, lr_fn=lambda t: 0.8, wd=0.01)
    assert worst["param"] <= Hn.TOL_PARAM


@pytest.mark.parametrize("variant", [None, "mfma_f32", "valu"])
def test_badly_scaled_weights_and_an_outlier_gradient(variant, monkeypatch):
    # Weights that are legal but nowhere near Glorot magnitude (rows of W1 / W2 200x and 50x larger or 10^4x smaller,
    # biases of order 10) and one gradient element 50 000 times the others in a million-element tensor: its normalized
    # gradient feature is ~1000 and its hidden pre-activations several 10^4. The default kernel carries the MLP's
    # operands as pairs of fp16 numbers; it must hold the same bar here as the fp32 kernels (no saturation at 65504,
    # no loss of the small rows). The other kernels are selected through the environment here (LOPT_APPLY fills in
    # a configuration field left at 0).
    if variant:
        monkeypatch.setenv("LOPT_APPLY", variant)
    cfg = Hn.make_cfg("small_fc_lopt")
    w = W.small_fc_weights_badly_scaled(3)

    class Outlier(Hn.Case):
        def grad(self, i, step):
            g = super().grad(i, step)
            if g.size > 1000:
                g[5 % g.shape[0], 7] = 50.0
            return g

    shapes = [(1024, 1024), (64, 256), (300,), (130, 260)]
    worst = Hn.run_free(Outlier(120, _specs(shapes)), cfg, w, 3, lr_fn=lambda t: 0.9, wd=0.01)
    print(f"badly scaled weights, LOPT_APPLY={variant}: worst {worst}")
    assert worst["param"] <= Hn.TOL_PARAM and worst["delta"] <= Hn.TOL_DELTA


def test_velo_vector_alu_variant_matches_the_oracle(monkeypatch):
    monkeypatch.setenv("LOPT_APPLY", "valu")
    cfg = Hn.make_cfg("velo")
    Hn.run_free(Hn.Case(106, W.config1_shapes(), "gauss_logscale"), cfg, W.velo_weights(1), 4, wd=0.01)


@pytest.mark.parametrize("kind", ["small_fc_lopt", "velo"])
def test_degenerate_gradients(kind):
    # an all-zero gradient, a constant gradient (rank one, zero variance), one huge outlier, tiny magnitudes
    cfg = Hn.make_cfg(kind)
    w = Hn.random_weights(cfg, 4)
    shapes = [(64, 256), (64, 256), (64, 256), (64, 256), (300,)]

    class Degenerate(Hn.Case):
        def grad(self, i, step):
            g = super().grad(i, step)
            if i == 0:
                g[:] = 0.0
            elif i == 1:
                g[:] = 3e-4
            elif i == 2:
                g[5, 7] = 50.0
            elif i == 3:
                g *= np.float32(1e-12)
            else:
                g[:] = 0.0
            return g

    worst = Hn.run_free(Degenerate(107, _specs(shapes)), cfg, w, 3)
    assert np.isfinite(worst["param"])


@pytest.mark.parametrize("kind", ["small_fc_lopt", "velo"])
def test_tiny_eps_acc_takes_the_library_reciprocal_roots(kind):
    # With eps_acc below 1e-30 the kernels must not use the bare reciprocal / reciprocal-square-root instructions
    # (they flush inputs below the smallest normal float): separate instantiations, exercised here with eps_acc = 0
    # and eps_acc = 1e-38 on gradients that keep every accumulator positive.
    for eps in (0.0, 1e-38):
        cfg = Hn.make_cfg(kind) if kind == "small_fc_lopt" else Hn.make_cfg(kind, lstm_hidden=32, n_bank=16)
        cfg.eps_acc = eps
        w = Hn.random_weights(cfg, 5)
        worst = Hn.run_free(Hn.Case(108, _specs([(130, 260), (64, 256), (300,), (70, 36)]), "gauss_logscale"), cfg, w, 3,
                            lr_fn=lambda t: 0.9, wd=0.01)
        assert worst["param"] <= Hn.TOL_PARAM


@pytest.mark.parametrize("tall", [[], [(6145, 2)]])
@pytest.mark.parametrize("kind,state_pass", [("small_fc_lopt", "apply"), ("small_fc_lopt", "stats"), ("velo", "apply"), ("velo", "stats")])
def test_narrow_rows_several_to_an_access(kind, state_pass, tall):
    # tensors of up to 128 columns: one column a lane, 64 / n rows to an access, one or two 64-column segments whose rows the wavefronts
    # share; row counts around the rows of an access and of a trip, on and off the 16-byte grid, short lists and (with a tensor of
    # more rows than those may have) the ordinary form. 129 to 131 columns beside them: a second tile of one to three columns.
    cfg = Hn.make_cfg(kind, state_pass=state_pass) if kind == "small_fc_lopt" else Hn.make_cfg(kind, lstm_hidden=32, n_bank=8, state_pass=state_pass)
    w = Hn.random_weights(cfg, seed=33)
    shapes = [(63, 1), (64, 1), (65, 1), (129, 1), (31, 2), (21, 3), (43, 3), (16, 4), (8, 8), (7, 9), (29, 9), (3, 21), (2, 32), (9, 32), (5, 33),
              (64, 33), (1, 63), (17, 64), (65, 64), (6, 65), (31, 100), (9, 127), (70, 128), (3, 129), (33, 130), (8, 131), (1, 7), (1, 128)] + tall
    assert plan(shapes, kind=kind, lstm_hidden=32, n_bank=8)["short_list"] == (not tall)
    worst = Hn.run_free(Hn.Case(133, _specs(shapes), "gauss_logscale"), cfg, w, 3, lr_fn=lambda t: 0.5, wd=0.01)
    assert worst["param"] <= Hn.TOL_PARAM


@pytest.mark.parametrize("tall", [[], [(6145, 2)]])
@pytest.mark.parametrize("kind", ["small_fc_lopt", "velo"])
def test_narrow_rows_over_several_trips(kind, tall):
    # tiles of 64 rows: every wavefront of the statistics pass (8 times 64 / n rows a trip, all four together) and, from 21 columns on, of VeLO's apply pass
    # (twice as many) makes more than one trip, the last tile of a tensor a ragged one. The columns of one element only make the list long enough
    # for such tiles.
    lstm = {} if kind == "small_fc_lopt" else dict(lstm_hidden=32, n_bank=8)
    wide = [(777, 9), (775, 13), (773, 21), (771, 27), (769, 33), (770, 61), (771, 64), (773, 65), (775, 101)]
    shapes = wide + [(6100, 1)] * 21 + tall
    r = plan(shapes, kind=kind, **lstm)
    assert r["short_list"] == (not tall)
    for (m, n), t in zip(wide, r["tensors"]):
        step = 8 * (64 // n if n <= 64 else 1) // (1 if n <= 64 else 2)
        assert t["TR"] == 64 > step and m % 64 and (n < 21 or 64 > 2 * step)
    cfg = Hn.make_cfg(kind, **lstm)
    worst = Hn.run_free(Hn.Case(137, _specs(shapes), "gauss_logscale"), cfg, Hn.random_weights(cfg, seed=39), 2, lr_fn=lambda t: 0.5, wd=0.01)
    assert worst["param"] <= Hn.TOL_PARAM


@pytest.mark.parametrize("hidden", [16, 32])
def test_rows_on_the_16_byte_grid_read_with_ordinary_loads_by_the_statistics_of_short_lists(hidden):
    # small_fc_lopt from 1.5 M elements on (VeLO at every size)
    shapes = [(1301, 1300), (65, 260), (7,)]
    assert plan(shapes, hidden=hidden)["keep_line"] == 1 and plan(shapes[1:], hidden=hidden)["keep_line"] == 0
    cfg = Hn.make_cfg("small_fc_lopt", hidden=hidden)
    worst = Hn.run_free(Hn.Case(138, _specs(shapes), "gauss_logscale"), cfg, Hn.random_weights(cfg, seed=40), 2, lr_fn=lambda t: 0.5, wd=0.01)
    assert worst["param"] <= Hn.TOL_PARAM


@pytest.mark.parametrize("rows,cols", [(13, n) for n in (1, 9, 63, 65, 127, 129, 255, 257, 258, 259, 515)] + [(2500, 2557)])
def test_velo_rows_off_the_grid_write_nothing_beside_the_tensor(rows, cols):
    # parameters and gradients between guard values: the last access of a row ends with the row, that of a tensor with the tensor
    import torch
    import paper_2506_10315_amd as P
    # (the last list is long enough for nontemporal accesses)
    cfg = Hn.make_cfg("velo", lstm_hidden=32, n_bank=8)
    assert plan([(rows, cols)], kind="velo", lstm_hidden=32, n_bank=8)["off_grid_nt"] == (rows > 13)
    n = rows * cols
    gen = torch.Generator(device="cuda:0").manual_seed(cols)
    flat = torch.randn(n + 128, device="cuda:0", generator=gen) * 0.02
    grad = torch.randn(n, device="cuda:0", generator=gen) * 1e-3
    before = flat.clone()
    opt = P.LearnedOptimizer(cfg, Hn.random_weights(cfg, seed=34), [(rows, cols)])
    opt.step([flat[64:64 + n].view(rows, cols)], [grad.view(rows, cols)], lr=1.0)
    torch.cuda.synchronize()
    assert torch.equal(flat[:64], before[:64]) and torch.equal(flat[64 + n:], before[64 + n:])
    assert float((flat[64:64 + n] != before[64:64 + n]).float().mean()) > 0.9


@pytest.mark.parametrize("kind,hidden", [("velo", 4), ("small_fc_lopt", 16), ("small_fc_lopt", 32)])
def test_rows_off_the_grid_with_either_kind_of_access_in_the_apply_pass(kind, hidden):
    # lists long enough for the apply pass to access rows off the 16-byte grid nontemporally (VeLO and width 16 from 6 and 7 M elements
    # on, width 32 from 7 to 13 M); shorter ones, with ordinary accesses, are everywhere above
    cfg = Hn.make_cfg(kind, hidden=hidden) if kind == "small_fc_lopt" else Hn.make_cfg(kind, lstm_hidden=32, n_bank=8)
    shapes = [(2700, 2731), (65, 258), (7,)]
    r = plan(shapes, kind=kind, hidden=hidden, lstm_hidden=32, n_bank=8)
    assert r["strip_ordinary"] == 0 if hidden == 32 else r["off_grid_nt"] == 1
    worst = Hn.run_free(Hn.Case(135, _specs(shapes), "gauss_logscale"), cfg, Hn.random_weights(cfg, seed=35), 1, lr_fn=lambda t: 0.5, wd=0.01)
    assert worst["param"] <= Hn.TOL_PARAM


RANGE_SHAPES = [(33, 131), (20, 259), (31, 100), (40, 7), (64, 256), (40, 132), (1, 1031)]   # off the 16-byte grid, narrow, on it, a vector


@pytest.mark.parametrize("tall", [[], [(6145, 2)]])
@pytest.mark.parametrize("kind,state_pass", [("small_fc_lopt", "apply"), ("small_fc_lopt", "stats"), ("velo", "apply")])
@pytest.mark.parametrize("scale", [2.5e-23, 1e-21, 1e-19, 1e9, 1e12])
def test_statistics_of_gradients_whose_squares_leave_the_fp32_range(scale, kind, state_pass, tall):
    # g sqrt(mean r / (r c)) is a number of ordinary size for gradients of any scale; g^2 is not. Each statistic that fp32 holds has to be
    # right, in short lists and (with a tensor of more rows than those may have) the ordinary form. Steps from zero state: M_1 = 0.1 g.
    # The first column and row are 100 times smaller than the rest.
    import torch
    import paper_2506_10315_amd as P
    from oracle import lopt_oracle as O
    lstm = {} if kind == "small_fc_lopt" else dict(lstm_hidden=32, n_bank=8)
    cfg = Hn.make_cfg(kind, state_pass=state_pass, **lstm)
    shapes = RANGE_SHAPES + tall
    assert plan(shapes, kind=kind, **lstm)["short_list"] == (not tall)
    ocfg, rng = Hn.oracle_config_from(cfg), np.random.default_rng(41)
    ps = [rng.standard_normal(s).astype(np.float32) * np.float32(0.02) for s in shapes]
    gs = [(rng.standard_normal(s) * scale).astype(np.float32) for s in shapes]
    for g in gs:
        g[0] *= np.float32(0.01) if g.shape[0] > 1 else np.float32(1)
        g[:, 0] *= np.float32(0.01)
    opt = P.LearnedOptimizer(cfg, Hn.random_weights(cfg, seed=36), shapes)
    new = [torch.from_numpy(p).cuda() for p in ps]
    opt.step(new, [torch.from_numpy(g).cuda() for g in gs], lr=1.0, loss=1.0)
    torch.cuda.synchronize()
    if kind == "small_fc_lopt":   # (a statistic beyond fp32 is an infinite input of the LSTM)
        assert all(bool(torch.isfinite(p).all()) for p in new)
    for i, got in enumerate(opt.stats()):
        st = O.init_state(*shapes[i], ocfg)
        O.update_accumulators(st, gs[i], ocfg)
        want = O.tensor_statistics(ps[i], gs[i], st, ocfg, 0)[:ocfg.n_normalized]
        rel = np.abs(got.cpu().numpy().astype(np.float64) - want) / (want + ocfg.eps_norm)
        # a sum of squares beyond fp32, or of values whose squares (those of r, c and V: fourth powers of g) are, is not held at all
        held = want * np.prod(shapes[i]) < 1e38
        assert held[6:13].all() and held[22:25].all()
        assert rel[held].max() <= Hn.TOL_STATS, (shapes[i], int(np.argmax(np.where(held, rel, 0.0))), rel[held].max())


@pytest.mark.parametrize("tall", [[], [(6145, 2)]])
@pytest.mark.parametrize("kind", ["small_fc_lopt", "velo"])
@pytest.mark.parametrize("eps", [1e-24, 1e-32])
def test_zero_gradients_with_a_small_eps_acc(eps, kind, tall):
    # a layer that gets no gradient: 1/(r+eps) and 1/(c+eps) are in the fp32 range, their product is not
    class Zeros(Hn.Case):
        def grad(self, i, step):
            return super().grad(i, step) * np.float32(0 if i % 2 == 0 else 1e-12)

    cfg = Hn.make_cfg(kind, **({} if kind == "small_fc_lopt" else dict(lstm_hidden=32, n_bank=8)))
    cfg.eps_acc = eps
    shapes = [s for s in RANGE_SHAPES for _ in range(2)] + tall
    worst = Hn.run_free(Zeros(136, _specs(shapes)), cfg, Hn.random_weights(cfg, seed=37), 2, lr_fn=lambda t: 0.5, wd=0.01)
    assert worst["param"] <= Hn.TOL_PARAM


@pytest.mark.parametrize("kind", ["small_fc_lopt", "velo"])
@pytest.mark.parametrize("copies", [1, 4])
def test_row_and_column_statistics_of_short_lists_are_sums_in_double(kind, copies):
    # mean(r_k^2) and mean(c_k^2) against the same of the fp32 r_k, c_k that the step has left. What remains is the rounding of the
    # statistic itself, 2^-24, and the products and sums in double; sums of 256 rows in fp32 go beyond it by up to 1e-7.
    import torch
    import paper_2506_10315_amd as P
    lstm = {} if kind == "small_fc_lopt" else dict(lstm_hidden=32, n_bank=8)
    cfg = Hn.make_cfg(kind, **lstm)
    shapes = [(256, 300), (200, 257), (131, 250), (1000, 40), (513, 512), (777, 9)] * copies
    assert plan(shapes, kind=kind, **lstm)["short_list"] == 1
    rng = np.random.default_rng(51)
    ps = [rng.standard_normal(s).astype(np.float32) for s in shapes]
    gs = [(rng.standard_normal(s) * np.exp(rng.standard_normal((s[0], 1)) + rng.standard_normal((1, s[1])))).astype(np.float32) for s in shapes]
    opt = P.LearnedOptimizer(cfg, Hn.random_weights(cfg, seed=38), shapes)
    opt.step([torch.from_numpy(p).cuda() for p in ps], [torch.from_numpy(g).cuda() for g in gs], lr=1.0, loss=1.0)
    torch.cuda.synchronize()
    worst = 0.0
    for i, got in enumerate(opt.stats()):
        v = opt.state_views(i)
        want = np.array([float((x.double() ** 2).mean()) for x in list(v["r"]) + list(v["c"])])
        worst = max(worst, float((np.abs(got[13:19].cpu().numpy().astype(np.float64) - want) / want).max()))
    print("worst", worst)
    assert worst <= 2.0 ** -24 * (1 + 1e-3)
