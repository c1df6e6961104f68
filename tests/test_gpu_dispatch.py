"""GPU tests of the size rules of the scoring kernels: the shapes on either side of a rule,
each against the fp64 oracle on every row at the acceptance bar.
"""
import numpy as np
import pytest
import torch

from oracle import olive_oracle as O
from paper_2609_36246_amd import _lib as L
from paper_2609_36246_amd import workloads as W
from tests.gpu_harness import compare, run_hip, say, to_np
from tests.test_gpu_backward import check_grads, oracle_backward, run_backward

pytestmark = pytest.mark.gpu

FORWARD = ("kl", "counts", "logp_s", "logp_t", "am_s", "am_t", "ce")


@pytest.fixture(scope="module", autouse=True)
def gpu():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    L.load()


def custom(name, seed=0, **kw):
    return W.make_workload(name, seed, device="cuda", spec=W.custom_spec(name=name, **kw))


# Few position tiles take more than 32 vocabulary splits (up to 256, one round of the
# grid). T = positions; at V = 40000 (157 vocabulary tiles) one 256-row tile gives 157
# splits, two 79 or 128, nine (256-row) 28: both sides of the rule. am ties: the first
# row's winner is copied to the last vocabulary entry, so that the winner's split and one
# of the last splits (past the first 32-split mask word) hold the exact tie.
@pytest.mark.parametrize("T,outs,narrow", [
    (1, "forward", False), (160, "forward", False), (256, "forward", True),
    (257, "forward", False), (2048, "forward", False), (2049, "forward", False),
    (130, "both", False), (200, "student", False), (300, "jsd", False)])
def test_few_positions_many_splits(T, outs, narrow):
    say("few positions", T, outs)
    V = 40000
    wl = custom("few%d" % T, num_seqs=1, seq_len=T, vocab=V, d_student=64, d_teacher=128,
                cut_rule=("frac", 0.0, 0.0))
    z = (wl["h_student"][:1].float() @ wl["w_student"].float())[0]
    j = int(torch.argmax(z))
    wl["w_student"][:, V - 1] = wl["w_student"][:, j]
    o = FORWARD + (("kl_rev",) if outs in ("both", "jsd") else ()) + \
        (("jsd",) if outs == "jsd" else ())
    hip = run_hip(wl, outputs=("logp_s", "am_s") if outs == "student" else o,
                  student_only=outs == "student", narrow=narrow)
    ns = hip["stats"]["splits"]
    assert hip["stats"]["kernel"] == "mfma"
    # (calls on the 256 x 128 kernel take 64 at most, as its top-K lists do)
    assert ns >= 64 if T <= 300 else ns <= 32, ns
    assert hip["stats"]["flagged"] >= 1 and hip["am_s"][0] == min(j, V - 1)
    compare(hip, wl, student_only=outs == "student", label="few-%d-%s" % (T, outs))


# The combine pass holds fewer registers from 8193 positions on, up to widths of 2048.
@pytest.mark.parametrize("T,ds,dt", [(8192, 64, 128), (8193, 64, 128), (8193, 128, 2112)])
@pytest.mark.parametrize("student", [False, True], ids=["both", "student"])
def test_combine_of_many_positions(T, ds, dt, student):
    say("combine", T, ds, dt, student)
    wl = custom("combine", num_seqs=1, seq_len=T, vocab=300, d_student=ds, d_teacher=dt,
                cut_rule=("frac", 0.2, 0.8), target_source="uniform")
    z = wl["h_student"][T - 1].float() @ wl["w_student"].float()
    j = int(torch.argmax(z))
    wl["w_student"][:, 299] = wl["w_student"][:, j]   # the last row ties exactly
    hip = run_hip(wl, student_only=student, outputs=("logp_s", "am_s") if student else FORWARD)
    assert hip["stats"]["flagged"] >= 1 and hip["am_s"][T - 1] == min(j, 299)
    compare(hip, wl, student_only=student, label="combine-%d-%d" % (T, dt))


def test_backward_of_few_rows_many_splits():
    say("backward of few rows")
    wl = custom("fewbw", num_seqs=2, seq_len=100, vocab=33000, d_student=128, d_teacher=64,
                cut_rule=("frac", 0.5, 0.5))
    T, B = wl["total_positions"], 2
    f = lambda t: to_np(t).astype(np.float64)   # noqa: E731
    for w_kl in (0.0, 0.5):
        ctx = L.olive_score_init(
            L.make_desc(33000, 128, 64, L.OLIVE_BF16, L.OLIVE_W_DV, 1.0, 1.0, max_positions=T,
                        max_seqs=B, flags=L.OLIVE_FLAG_BACKWARD), wl["w_student"], wl["w_teacher"])
        gh = torch.full((T, 128), float("nan"), device="cuda")
        gw = torch.full((128, 33000), float("nan"), device="cuda")
        batch = L.make_batch(wl["cu_seqlens"], wl["cut"], wl["targets"], wl["h_student"],
                             wl["h_teacher"], wl["valid_len"])
        L.olive_score_backward(ctx, batch, L.make_grad_outputs(1.0, w_kl, gh, gw))
        torch.cuda.synchronize()
        L.olive_score_free(ctx)
        ref = O.backward(f(wl["h_student"]), f(wl["w_student"]), to_np(wl["targets"]),
                         to_np(wl["cu_seqlens"]), to_np(wl["cut"]), None, f(wl["h_teacher"]),
                         f(wl["w_teacher"]), w_ce=1.0, w_kl=w_kl)
        # bf16 rounding of g and its fp32 exponentials (2^-8), fp32 accumulation (K 2^-24)
        ga, ha, wa = np.abs(ref["g"]), np.abs(f(wl["h_student"])), np.abs(f(wl["w_student"]))
        bh = (2.0 ** -8 + 33000 * 2.0 ** -24) * (ga @ wa.T) + 1e-6
        bw = (2.0 ** -8 + T * 2.0 ** -24) * (ha[ref["rows"]].T @ ga) + 1e-6
        assert np.all(np.abs(to_np(gh)[ref["rows"]] - ref["grad_h"][ref["rows"]]) <= bh)
        assert np.all(np.abs(to_np(gw) - ref["grad_w"]) <= bw)


# The products (tiles of 256 x 256) split K over more units where their tiles leave compute
# units idle: dL/dh of one tile with few K steps (none) and more (up to a part per step),
# ragged tiles in both directions, a tile count that fits no second part evenly, two chunks of
# rows (the second one short); dL/dW of one and of several tiles, both layouts, an odd V, on
# a second chunk, and one K step (no part). The parts add in a fixed order: repeated calls
# are bit-identical.
@pytest.mark.parametrize("T,ds,V", [(1, 64, 300), (129, 320, 20000), (700, 576, 3000),
                                    (2900, 64, 1000), (8200, 128, 300), (5000, 64, 257),
                                    (8900, 320, 1001), (60, 64, 4000)])
@pytest.mark.parametrize("layout", [L.OLIVE_W_DV, L.OLIVE_W_VD], ids=["dv", "vd"])
def test_backward_product_splits(T, ds, V, layout):
    say("backward product", T, ds, V, layout)
    wl = custom("parts", num_seqs=1, seq_len=T, vocab=V, d_student=ds, d_teacher=64,
                cut_rule=("frac", 0.0, 0.0))
    dv = layout == L.OLIVE_W_DV   # (run_backward drops the [V][d] weights a context borrows)
    hip = run_backward(wl, keep_ctx=dv, layout=layout)
    if dv:
        again = run_backward(wl, ctx=hip["ctx"])
        L.olive_score_free(hip["ctx"])
        for k in ("h", "w"):
            np.testing.assert_array_equal(hip[k], again[k], err_msg=k)
    check_grads(hip, oracle_backward(wl, 1.0, 0.0, O.REGION_TEACHER), wl, "product-%d" % T)


# dL/dW with more 256 x 256 tiles than compute units (274 x 2): a workgroup's pipeline goes on
# into its next tile, with one K step a tile (A's prefetch two tiles ahead) and with three,
# whole tiles and ragged ones, values stored one by one (odd V, [d][V]) and in fours.
@pytest.mark.parametrize("T,V", [(40, 70001), (40, 70000), (150, 70001)])
@pytest.mark.parametrize("layout", [L.OLIVE_W_DV, L.OLIVE_W_VD], ids=["dv", "vd"])
def test_backward_product_units_follow_each_other(T, V, layout):
    say("backward product, several units a workgroup", T, V, layout)
    wl = custom("units", num_seqs=1, seq_len=T, vocab=V, d_student=320, d_teacher=64,
                cut_rule=("frac", 0.0, 0.0), target_source="uniform")
    hip = run_backward(wl, layout=layout)
    check_grads(hip, oracle_backward(wl, 1.0, 0.0, O.REGION_TEACHER), wl, "units-%d" % T)


# The same onto C: a second chunk of rows (8 past 8192) adds to 36 x 8 tiles, the loads of C
# behind the next tile's prefetches. Sampled columns and rows against the oracle.
def test_backward_product_units_add_a_second_chunk():
    say("backward product, several units a workgroup, second chunk")
    T, V, ds = 8200, 9001, 2048
    wl = custom("units2", num_seqs=1, seq_len=T, vocab=V, d_student=ds, d_teacher=64,
                cut_rule=("frac", 0.0, 0.0), target_source="uniform")
    rng = np.random.default_rng(5)
    cols = np.unique(np.concatenate([[0, 255, 256, V - 1], rng.choice(V, 60, replace=False)]))
    rows = np.unique(np.concatenate([[0, 8191, 8192, T - 1], rng.choice(T, 28, replace=False)]))
    f64 = lambda t: to_np(t).astype(np.float64)   # noqa: E731
    hs, ws, y = f64(wl["h_student"]), f64(wl["w_student"]), to_np(wl["targets"])
    # the logit gradients of every row: p - onehot(y)
    z = hs @ ws
    z -= z.max(axis=1, keepdims=True)
    np.exp(z, out=z)
    z /= z.sum(axis=1, keepdims=True)
    z[np.arange(T), y] -= 1.0
    ref = {"rows": np.arange(T), "in_region": np.ones(T, dtype=bool), "g": z,
           "grad_w": hs.T @ z[:, cols], "grad_h": np.zeros((T, ds))}
    ref["grad_h"][rows] = z[rows] @ ws.T
    for layout in (L.OLIVE_W_DV, L.OLIVE_W_VD):
        hip = run_backward(wl, layout=layout)
        check_grads({"w": hip["w"]}, ref, wl, "units2-w-%d" % layout, cols=cols)
        check_grads({"h": hip["h"]}, ref, wl, "units2-h-%d" % layout, rows=rows)


# dL/dW of few tiles (three here) runs on as many compute units as dL/dh: over 9000 rows the
# two gradients alone take about as long (145 and 130 us; 282 with dL/dW on three).
def test_backward_products_of_few_tiles_fill_the_chip():
    say("backward products of few tiles")
    wl = custom("fewtiles", num_seqs=1, seq_len=9000, vocab=600, d_student=64, d_teacher=64,
                cut_rule=("frac", 0.0, 0.0))
    ctx = run_backward(wl, keep_ctx=True)["ctx"]
    batch = L.make_batch(wl["cu_seqlens"], wl["cut"], wl["targets"], wl["h_student"],
                         wl["h_teacher"], wl["valid_len"])
    gh, gw = torch.empty(9000, 64, device="cuda"), torch.empty(64, 600, device="cuda")
    grads = {"h": L.make_grad_outputs(1.0, 0.0, gh, None),
             "w": L.make_grad_outputs(1.0, 0.0, None, gw)}
    best = dict.fromkeys(grads, 1e9)
    for _ in range(10):
        for k, g in grads.items():
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(10):
                L.olive_score_backward(ctx, batch, g)
            b.record()
            b.synchronize()
            best[k] = min(best[k], a.elapsed_time(b) * 100.0)
    L.olive_score_free(ctx)
    say("dL/dh alone %.0f us, dL/dW alone %.0f us" % (best["h"], best["w"]))
    assert best["w"] < 1.4 * best["h"], best


# The workspace of the dL/dh product is no larger than its splits use.
def test_small_backward_context_is_small():
    say("memory of a small backward context")
    wl = custom("small-bw", num_seqs=1, seq_len=64, vocab=1000, d_student=64, d_teacher=64,
                cut_rule=("frac", 0.0, 0.0))
    run_backward(wl)   # the library's code and the runtime's own memory are loaded
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    ctx = L.olive_score_init(
        L.make_desc(1000, 64, 64, L.OLIVE_BF16, L.OLIVE_W_DV, max_positions=64, max_seqs=1,
                    flags=L.OLIVE_FLAG_BACKWARD), wl["w_student"], wl["w_teacher"])
    used = before - torch.cuda.mem_get_info()[0]
    L.olive_score_free(ctx)
    say("%.1f MB" % (used / 1e6))
    assert used < 64e6, used


# The generic kernel's tiles: 128 vocabulary rows x 64 positions, K in steps of 32 read in
# groups of 4 elements where width and alignment allow; edges and remainders of each.
@pytest.mark.parametrize("dtype,T,V,ds,dt,off", [
    ("f32", 1, 1, 1, 1, 0), ("f32", 64, 128, 32, 64, 0), ("f32", 65, 129, 33, 31, 0),
    ("f32", 63, 255, 36, 100, 0), ("f32", 130, 20001, 40, 8, 0), ("f32", 700, 300, 5, 67, 1),
    ("bf16", 70, 200, 64, 64, 0), ("bf16", 65, 1000, 36, 12, 0), ("bf16", 129, 700, 33, 96, 0),
    ("bf16", 40, 5000, 128, 64, 1)])
def test_generic_kernel_tile_edges(dtype, T, V, ds, dt, off):
    say("generic tiles", dtype, T, V, ds, dt, "offset", off)
    wl = custom("generic", num_seqs=1, seq_len=T, vocab=V, d_student=ds, d_teacher=dt,
                dtype=dtype, cut_rule=("frac", 0.0, 0.0), target_source="uniform")
    if off:   # hidden rows one element off the loads' alignment
        for k in ("h_student", "h_teacher"):
            b = torch.empty(wl[k].numel() + off, dtype=wl[k].dtype, device="cuda")
            b[off:] = wl[k].reshape(-1)
            wl[k] = b[off:].view(wl[k].shape)
    hip = run_hip(wl, outputs=FORWARD + ("kl_rev",))
    assert hip["stats"]["kernel"] == "generic"
    compare(hip, wl, label="generic-%s-%d-%d" % (dtype, T, V))
    alone = run_hip(wl, outputs=("logp_s", "am_s"), student_only=True)
    compare(alone, wl, student_only=True, label="generic-student")


# Widths up to 8 run one group of 8 K elements a step.
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("T,V,ds,dt", [(70, 300, 8, 8), (65, 129, 7, 4), (64, 128, 9, 8),
                                       (130, 1001, 8, 9), (1, 1, 2, 8)])
def test_generic_kernel_narrow_widths(dtype, T, V, ds, dt):
    say("generic widths", dtype, T, V, ds, dt)
    wl = custom("narrow", num_seqs=1, seq_len=T, vocab=V, d_student=ds, d_teacher=dt,
                dtype=dtype, cut_rule=("frac", 0.0, 0.0), target_source="uniform")
    hip = run_hip(wl, outputs=FORWARD + ("kl_rev",))
    assert hip["stats"]["kernel"] == "generic"
    compare(hip, wl, label="widths-%s-%d-%d" % (dtype, ds, dt))
    alone = run_hip(wl, outputs=("logp_s", "am_s"), student_only=True)
    compare(alone, wl, student_only=True, label="widths-student")


def test_generic_kernel_nan_and_infinite_rows_stay_their_own():
    say("generic kernel, rows with NaN and infinite hidden states")
    wl = custom("generic-nan", num_seqs=1, seq_len=70, vocab=300, d_student=33, d_teacher=64,
                dtype="f32", cut_rule=("frac", 0.0, 0.0), target_source="uniform")
    clean = run_hip(wl, outputs=FORWARD)
    wl["h_student"][3, 5] = float("nan")
    wl["h_student"][66, 7] = float("inf")
    hip = run_hip(wl, outputs=FORWARD)
    assert np.all(np.isnan(hip["logp_s"][[3, 66]])) and np.all(np.isnan(hip["kl"][[3, 66]]))
    keep = np.setdiff1d(np.arange(70), [3, 66])
    for k in ("logp_s", "logp_t", "kl", "am_s", "am_t"):
        np.testing.assert_array_equal(hip[k][keep], clean[k][keep], err_msg=k)
    np.testing.assert_array_equal(hip["logp_t"], clean["logp_t"])


# Infinite logits of the generic kernel (rows 10 and 11 are one lane's, 200 another's): two of
# +inf leave no normaliser, wherever they lie, one has all the weight; those of -inf have none.
@pytest.mark.parametrize("rows", [(10,), (10, 11), (10, 200), (10, 11, 40, 299)])
def test_generic_kernel_infinite_logits(rows):
    say("generic kernel, infinite logits", rows)
    V, d, T = 300, 33, 3
    g = torch.Generator(device="cuda").manual_seed(3)
    w = torch.randn(V, d, generator=g, device="cuda")
    w[:, 0] = 0.0
    h = torch.zeros(T, d, device="cuda")
    h[:, 0], h[:, 1] = 1e20, 1.0
    cu, cut, y = (torch.tensor(x, dtype=torch.int32, device="cuda")
                  for x in ([0, T], [0], [0, 100, 298]))
    desc = L.make_desc(V, d, 0, L.OLIVE_F32, L.OLIVE_W_VD, 1.0, max_positions=T, max_seqs=1)
    for sign in (1.0, -1.0):
        w[list(rows), 0] = sign * 1e30
        logp = torch.zeros(T, device="cuda")
        ctx = L.olive_score_init(desc, w)
        L.olive_token_logprobs(ctx, L.make_batch(cu, cut, y, h), logp)
        torch.cuda.synchronize()
        L.olive_score_free(ctx)
        if sign > 0:
            want = -np.inf if len(rows) == 1 else np.nan
            np.testing.assert_array_equal(to_np(logp), np.full(T, want, dtype=np.float32))
        else:
            z = to_np(w[:, 1]).astype(np.float64)
            keep = np.setdiff1d(np.arange(V), rows)
            np.testing.assert_allclose(to_np(logp), z[[0, 100, 298]] - np.logaddexp.reduce(z[keep]),
                                       atol=1e-5)


# The generic path's exact re-decision cuts its vocabulary chunks by the flagged rows'
# count: 1 row, a batch and one more (8 parts a chunk), and enough for whole chunks.
@pytest.mark.parametrize("dtype,ties", [("f32", 1), ("f32", 9), ("bf16", 9), ("f32", 400)])
def test_generic_exact_decision_parts(dtype, ties):
    say("generic re-decision", dtype, ties)
    V, T = 20003, 420
    wl = custom("parts", num_seqs=1, seq_len=T, vocab=V, d_student=72, d_teacher=33, dtype=dtype,
                cut_rule=("frac", 0.0, 0.0), target_source="uniform")
    z = wl["h_student"][:ties].float() @ wl["w_student"].float()
    for j in sorted(set(torch.argmax(z, dim=1).tolist())):
        wl["w_student"][:, (j + V // 2) % V] = wl["w_student"][:, j]   # an exact tie
    hip = run_hip(wl, outputs=FORWARD)
    assert hip["stats"]["kernel"] == "generic" and hip["stats"]["flagged"] >= min(ties, 300)
    compare(hip, wl, label="parts-%s-%d" % (dtype, ties))


# A call without a context forms its weight norms itself: in the scoring pass (in vocabulary
# tile t from the units of position tile t mod their number; V = 3001 shifts the last tile),
# or after it for the models with flagged rows (generic kernel). Rows 0 and T - 1 tie exactly,
# which decides by theta's own slack; the norms decide in the test after the next.
@pytest.mark.parametrize("simple", [False, True], ids=["mfma", "generic"])
@pytest.mark.parametrize("T,V,scales", [(1, 256, (1.0, 1.0)), (130, 3001, (1.0, 1.0)),
                                        (300, 40000, (2.0, 0.75))])
def test_static_call_forms_its_own_norms(T, V, scales, simple):
    say("static norms", T, V, scales, simple)
    wl = custom("norms", num_seqs=1, seq_len=T, vocab=V, d_student=64, d_teacher=192,
                cut_rule=("frac", 0.0, 0.0), target_source="uniform")
    wl["scale_student"], wl["scale_teacher"] = scales
    wl["w_teacher"][:, V - 1] *= 30.0   # the largest norm in the last row
    for m in ("student", "teacher"):
        h, w = wl["h_" + m], wl["w_" + m]
        for r in (0, T - 1):
            j = int(torch.argmax(h[r].float() @ w.float()))
            w[:, (j + V // 3) % V] = w[:, j]
    vd = [wl["w_" + m].t().contiguous() for m in ("student", "teacher")]
    o = {k: torch.full((T,), float("nan"), device="cuda") for k in ("kl", "logp_s", "logp_t")}
    o.update({k: torch.full((T,), -7, dtype=torch.int32, device="cuda") for k in ("am_s", "am_t")})
    desc = L.make_desc(V, 64, 192, L.OLIVE_BF16, L.OLIVE_W_VD, *scales, max_positions=T, max_seqs=1,
                       flags=L.OLIVE_FLAG_SIMPLE_KERNEL if simple else 0)
    batch = L.make_batch(wl["cu_seqlens"], wl["cut"], wl["targets"], wl["h_student"],
                         wl["h_teacher"], wl["valid_len"])
    for _ in range(2):
        L.olive_kl_masked_static(desc, vd[0], vd[1], batch, o["kl"], None, o["logp_s"],
                                 o["logp_t"], o["am_s"], o["am_t"])
    torch.cuda.synchronize()
    compare({k: to_np(v) for k, v in o.items()}, wl, label="static-%d-%d" % (T, V))


# Without greedy outputs a call without a context forms no norms: the other outputs are those of
# the call with them, in the time of a context's call (whose scoring kernel is the same then;
# with the norms the call took 78.5 us, without 67.5, as the context).
def test_static_call_without_greedy_outputs():
    say("static call without greedy outputs")
    T, V, ds, dt = 100, 16384, 1024, 2048
    wl = custom("nogreedy", num_seqs=1, seq_len=T, vocab=V, d_student=ds, d_teacher=dt,
                cut_rule=("frac", 0.3, 0.3), target_source="uniform")
    vd = [wl["w_" + m].t().contiguous() for m in ("student", "teacher")]
    batch = L.make_batch(wl["cu_seqlens"], wl["cut"], wl["targets"], wl["h_student"],
                         wl["h_teacher"], wl["valid_len"])
    o = [{k: torch.full((T,), float("nan"), device="cuda") for k in ("kl", "logp_s", "logp_t")}
         for _ in range(3)]
    am = [torch.full((T,), -7, dtype=torch.int32, device="cuda") for _ in range(2)]
    desc = L.make_desc(V, ds, dt, L.OLIVE_BF16, L.OLIVE_W_VD, max_positions=T, max_seqs=1)
    narrow = L.make_desc(V, ds, dt, L.OLIVE_BF16, L.OLIVE_W_VD, max_positions=T, max_seqs=1,
                         flags=L.OLIVE_FLAG_NARROW_TILE)
    ctx = L.olive_score_init(narrow, vd[0], vd[1])
    static = lambda x, *am: L.olive_kl_masked_static(   # noqa: E731
        desc, vd[0], vd[1], batch, x["kl"], None, x["logp_s"], x["logp_t"], *am)
    static(o[0], am[0], am[1])
    calls = {"static": lambda: static(o[1]), "context": lambda: L.olive_kl_masked(
        ctx, batch, o[2]["kl"], None, o[2]["logp_s"], o[2]["logp_t"])}
    best = dict.fromkeys(calls, 1e9)
    for _ in range(20):
        for k, call in calls.items():
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(10):
                call()
            b.record()
            b.synchronize()
            best[k] = min(best[k], a.elapsed_time(b) * 100.0)
    L.olive_score_free(ctx)
    say("static %.1f us, context %.1f us" % (best["static"], best["context"]))
    for x in o[1:]:
        for k in x:
            np.testing.assert_array_equal(to_np(x[k]), to_np(o[0][k]), err_msg=k)
    assert best["static"] < 1.08 * best["context"], best


# Near ties that the weight norms decide: the exact winner's terms are B, s .. s, -B, so that
# its fp32 logit loses the s beside B and falls below theta, the lower bound of the maximum
# that the fp32 winner (all terms 0.75 s) sets with its own small rounding bound; only
# delta = d 2^-23 |h| max |w| with the winner's own norm takes it in. The other columns stay
# below both. The winner is the one row with a large norm, in the first, a middle or the
# (shifted) last vocabulary tile, of one and of three position tiles; 2^-90 scales it to
# where the squares of its weights underflow.
def norm_pair(V, d, winner, rival, scale):
    big, s = 2.0 ** 10, 2.0 ** -22
    w = torch.full((V, d), -0.2 / d, dtype=torch.float64)
    w[winner] = s
    w[winner, 0], w[winner, -1] = big, -big
    w[rival] = 0.75 * s
    w = (w * scale).to(torch.bfloat16)
    # the decision is the norm's: the winner's fp32 logit, in K order and in blocks of 16,
    # lies below theta and below what the other rows' norms allow, not below the bound
    z = w.double().sum(dim=1)
    assert int(z.argmax()) == winner
    norm = w.double().norm(dim=1)
    other = torch.cat([norm[:winner], norm[winner + 1:]]).max()
    slack = d * 2.0 ** -23
    theta = float(z[rival] * (1 - slack))
    x = w[winner].float()
    for parts in (x, x.reshape(-1, 16).double().sum(dim=1)):
        acc = np.float32(0)
        for v in parts.tolist():
            acc = np.float32(acc + v)
        assert theta - slack * d ** 0.5 * float(norm[winner]) < acc < \
            theta - slack * d ** 0.5 * float(other)
    return w


@pytest.mark.parametrize("kind", ["static", "static-generic", "context"])
@pytest.mark.parametrize("T,ws,wt", [(1, 0, 2), (300, 1, 0), (300, 2, 1)])
@pytest.mark.parametrize("exponent", [0, -90])
def test_weight_norms_decide_near_ties(kind, T, ws, wt, exponent):
    say("norms decide", kind, T, ws, wt, exponent)
    V, ds, dt = 3001, 64, 192
    winner = (5, 1500, 2999)   # the last tile holds rows 2745 .. 3000
    w = [norm_pair(V, d, winner[k], r, 2.0 ** exponent).cuda()
         for d, k, r in ((ds, ws, 700), (dt, wt, 2000))]
    h = [torch.ones(T, d, dtype=torch.bfloat16, device="cuda") for d in (ds, dt)]
    cu, cut, y = (torch.tensor(x, dtype=torch.int32, device="cuda") for x in ([0, T], [0], [0] * T))
    batch = L.make_batch(cu, cut, y, h[0], h[1], None)
    kl = torch.empty(T, device="cuda")
    am = [torch.full((T,), -7, dtype=torch.int32, device="cuda") for _ in range(2)]
    desc = L.make_desc(V, ds, dt, L.OLIVE_BF16, L.OLIVE_W_VD, 1.0, 1.0, max_positions=T, max_seqs=1,
                       flags=L.OLIVE_FLAG_SIMPLE_KERNEL if kind == "static-generic" else 0)
    if kind == "context":
        ctx = L.olive_score_init(desc, w[0], w[1])
        L.olive_kl_masked(ctx, batch, kl, None, None, None, am[0], am[1])
        torch.cuda.synchronize()
        L.olive_score_free(ctx)
    else:
        L.olive_kl_masked_static(desc, w[0], w[1], batch, kl, None, None, None, am[0], am[1])
        torch.cuda.synchronize()
    for m, k in ((0, ws), (1, wt)):
        np.testing.assert_array_equal(to_np(am[m]), np.full(T, winner[k], dtype=np.int32))


# Top-K lists of more splits than 32 (few position tiles, up to 64) and their selection.
@pytest.mark.parametrize("T", [1, 100, 400])
def test_topk_with_many_splits(T):
    say("top-K, many splits", T)
    wl = custom("tkfew%d" % T, num_seqs=1, seq_len=T, vocab=30000, d_student=64, d_teacher=128,
                cut_rule=("frac", 0.0, 0.0))
    o = FORWARD + ("kl_rev",)
    hip = run_hip(wl, outputs=o + ("overlap", "kl_topk", "tk_s", "tk_t"))
    assert 32 < hip["stats"]["splits"] <= 64
    compare(hip, wl, label="topk-splits-%d" % T)
    z = [to_np(wl["h_" + m]).astype(np.float64) @ to_np(wl["w_" + m]).astype(np.float64)
         for m in ("student", "teacher")]
    for k, zz in (("tk_s", z[0]), ("tk_t", z[1])):
        np.testing.assert_array_equal(hip[k], [O.topk_set(r, 16) for r in zz])
    plain = run_hip(wl, outputs=o)
    for k in ("kl", "kl_rev", "logp_s", "logp_t", "am_s", "am_t"):
        np.testing.assert_array_equal(hip[k], plain[k], err_msg=k)


# The greedy re-decision on the MFMA path: exact ties of the teacher's winner with up to 64
# candidates (decided from the queue), with more (the exhaustive scan, a workgroup each), on
# rows that fill a workgroup's four wavefronts, fewer and more.
@pytest.mark.parametrize("ties,T", [(2, 1), (3, 9), (64, 5), (65, 1), (300, 3), (300, 9)])
@pytest.mark.parametrize("narrow", [False, True], ids=["wide", "narrow"])
def test_greedy_ties_beyond_the_queue(ties, T, narrow):
    say("greedy ties", ties, T, narrow)
    V = 3001
    wl = custom("ties", num_seqs=1, seq_len=T, vocab=V, d_student=64, d_teacher=128,
                cut_rule=("frac", 0.0, 0.0), target_source="uniform")
    base = wl["h_teacher"][:1].clone()
    wl["h_teacher"][:] = base + 0.125 * wl["h_teacher"]
    cols = torch.arange(ties, device="cuda") * (V // ties) + V // ties - 1
    wl["w_teacher"][:, cols] = 0.5 * base.t()   # logits near |base|^2 / 2, the rest near N(0, 1)
    hip = run_hip(wl, narrow=narrow)
    assert hip["stats"]["kernel"] == "mfma" and hip["stats"]["flagged"] >= T
    np.testing.assert_array_equal(hip["am_t"], np.full(T, int(cols[0]), dtype=np.int32))
    compare(hip, wl, label="ties-%d-%d" % (ties, T))


# Exhaustive scans of several pairs run side by side: 8 rows with 300 tied columns each take
# about as long as one (a scan is all of such a call's time: 6.4 ms here; in turn on two
# compute units they took 24 ms).
def test_exhaustive_scans_run_side_by_side():
    say("exhaustive scans side by side")
    V, T = 32000, 64
    took = {}
    for rows in (1, 8):
        wl = custom("scans", num_seqs=1, seq_len=T, vocab=V, d_student=64, d_teacher=1024,
                    cut_rule=("frac", 0.0, 0.0), target_source="uniform")
        h = wl["h_teacher"].float()
        base = h[0] / h[0].norm()
        h -= (h @ base)[:, None] * base + 2.0 * base    # -2 along base, the tied rows +32
        h[:rows] += 34.0 * base
        wl["h_teacher"].copy_(h.to(torch.bfloat16))
        cols = torch.arange(300, device="cuda") * (V // 300) + 7
        wl["w_teacher"][:, cols] = (0.5 * base).to(torch.bfloat16)[:, None]
        hip = run_hip(wl, keep_ctx=True)
        np.testing.assert_array_equal(hip["am_t"][:rows], np.full(rows, 7, dtype=np.int32))
        assert rows <= hip["stats"]["flagged"] <= rows + 4
        best = []
        for _ in range(5):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            run_hip(wl, ctx=hip["ctx"], outputs=("logp_s", "am_t"))
            b.record()
            b.synchronize()
            best.append(a.elapsed_time(b))
        took[rows] = min(best)
        L.olive_score_free(hip["ctx"])
    say("one scan %.2f ms, eight %.2f ms" % (took[1], took[8]))
    assert took[8] < 2.0 * took[1], took
