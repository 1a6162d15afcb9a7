"""Whole-net parity on the GPU: the DPRS-selected path and the fixed paths of
the synthetic workloads against the chained float64 oracle (every layer
output rounded to the run dtype), the DP path on the measured cost table
against exhaustive enumeration, full-size sampled checks at the benchmark's
shapes, and HIP-graph replay."""

import numpy as np
import pytest

from oracle import numeric as O
from oracle.select import blockwise, exhaustive, problem_from_costs
from paper_2110_06037_amd import build_from_spec, native as N
from tests.gpu_util import TOL, err, from_dev, to_dev
from workloads import (CONV_SWEEP_SHAPES, conv_sweep, decode, fuse_projection, fuse_residual, generate, materialise,
                       mobilenet_v2, resnet18, resnet50, tiny_chain, to_f64, vgg16, with_batch)

pytestmark = pytest.mark.gpu


def decoded(t, dtype):
    return decode(t, dtype)


def oracle_out(spec, t, images=None):
    d = decoded(t, spec["dtype"])
    s = spec
    if images is not None:
        d["x"] = d["x"][:images]
        s = with_batch(spec, images)
    out = O.forward(s, d, storage="dtype")[-1]
    return out.reshape(out.shape[0], -1)


def run_out(g, spec, t):
    import torch
    xd = to_dev(t["x"], spec["dtype"])
    y = g.run(xd)
    torch.cuda.synchronize()
    return from_dev(y, spec["dtype"]).reshape(spec["batch"], -1), xd


def test_tiny_chain_measured_table_dp_equals_exhaustive_and_parity():
    spec = tiny_chain()
    t = generate(spec)
    g = build_from_spec(spec, t)
    g.profile(warmup=3, reps=10)
    costs = g.costs()
    for l in costs["layers"][1:-1]:
        assert all(r["ns"] > 0 for r in l["routines"]), l
    g.select("dprs")
    ids, total = g.path()
    tt, tup, count = exhaustive(problem_from_costs(costs))
    assert tuple(ids) + (0,) == tup and total == tt
    ref = oracle_out(spec, t)
    out, xd = run_out(g, spec, t)
    assert err(out, ref, "f32") <= TOL["f32"]
    # the timed run repeats every layer's launches; its result is the same bits
    y, ms = g.run_timed(xd, reps=3)
    assert np.array_equal(from_dev(y, "f32").reshape(spec["batch"], -1), out)
    assert ms[0] == 0 and all(m > 0 for m in ms[1:]), ms
    # cache-cold timing: a scratch buffer is written before each layer; the
    # result is unchanged
    g.set_option(N.OPT_FLUSH, 64 << 20)
    y, ms = g.run_timed(xd, reps=1)
    g.set_option(N.OPT_FLUSH, 0)
    assert np.array_equal(from_dev(y, "f32").reshape(spec["batch"], -1), out)
    assert ms[0] == 0 and all(m > 0 for m in ms[1:]), ms
    for lay in ("NCHW", "NHWC"):
        for algo in ("direct", "igemm"):
            g.select("fixed", lay, algo)
            out, _ = run_out(g, spec, t)
            assert err(out, ref, "f32") <= TOL["f32"], (lay, algo)
    # cache-cold unit profiling (median of single runs after a flush): a
    # complete positive cost table, cached apart from the warm one (so a warm
    # profile afterwards gives back the warm table), and its DP path is again
    # the exhaustive optimum of that table and matches the oracle
    g.set_option(N.OPT_FLUSH, 64 << 20)
    g.profile(warmup=1, reps=5)
    g.set_option(N.OPT_FLUSH, 0)
    cold = g.costs()
    for l in cold["layers"][1:-1]:
        assert all(r["ns"] > 0 for r in l["routines"]), l
    g.select("dprs")
    ids, total = g.path()
    tt, tup, _ = exhaustive(problem_from_costs(cold))
    assert tuple(ids) + (0,) == tup and total == tt
    out, _ = run_out(g, spec, t)
    assert err(out, ref, "f32") <= TOL["f32"]
    g.profile(warmup=3, reps=10)
    assert g.costs() == costs


@pytest.mark.parametrize("name", ["tiny", "mobilenetv2"])
def test_integrated_profiling_selects_the_measured_fastest_candidate(name):
    spec = tiny_chain() if name == "tiny" else mobilenet_v2(1)
    t = generate(spec)
    g = build_from_spec(spec, t)
    g.profile(warmup=2, reps=5)
    g.select("dprs")
    dp_ids, dp_t = g.path()
    cands = g.profile_integrated(warmup=2, reps=5)
    print(name, [(c["kind"], c["a"], c["b"], c["model_ns"], c["measured_ns"]) for c in cands],
          flush=True)
    assert cands[0]["kind"] == "dprs" and cands[0]["path"] == dp_ids and cands[0]["model_ns"] == dp_t
    assert all(c["measured_ns"] > 0 for c in cands)
    best = min(range(len(cands)), key=lambda i: (cands[i]["measured_ns"], i))
    ids, total = g.path()
    assert ids == cands[best]["path"] and total == cands[best]["model_ns"]
    out, _ = run_out(g, spec, t)
    assert err(out, oracle_out(spec, t), spec["dtype"]) <= TOL[spec["dtype"]]
    g.close()


def test_in_path_refinement_keeps_schemas_and_parity():
    # in-path refinement swaps a layer's routine only for one of the same
    # schema whose unit-profiled time is within the tolerance of the selected
    # one's, so the adapts stay as they were and the output still matches the
    # oracle
    spec = fuse_projection(fuse_residual(resnet50(2, "bf16")))
    t = generate(spec)
    g = build_from_spec(spec, t)
    g.profile(warmup=2, reps=5)
    g.select("dprs")
    before, _ = g.path()
    n = g.refine_in_path(tol_permille=200, max_alts=3, reps=5)
    after, total = g.path()
    changed = [i for i in range(len(after)) if after[i] != before[i]]
    print("refined layers", changed, [g.routines(i)[after[i]]["name"] for i in changed], flush=True)
    assert n == len(changed)
    for i in changed:
        r0, r1 = g.routines(i)[before[i]], g.routines(i)[after[i]]
        assert r1["schema"] == r0["schema"]
        assert r1["cost_ns"] <= r0["cost_ns"] * 1.2 + 1
    out, _ = run_out(g, spec, t)
    assert err(out, oracle_out(spec, t), spec["dtype"]) <= TOL[spec["dtype"]]
    g.close()


def test_in_path_refinement_times_the_launches_of_a_run():
    # a routine that computes the addition after its convolution against one
    # that is faster on the convolution alone, by less than an addition's
    # launch takes: swapping it in would add that launch to every run.  The
    # slow first layer gives the refined path a clear gain in either case, so
    # the end-to-end comparison does not undo the second layer's swap
    from paper_2110_06037_amd import Graph
    rng = np.random.default_rng(5)
    g = Graph("bf16", 8, 256, 14, 14, device=0, layouts=["NCHW", "NHWC"], algos=["direct", "igemm"])
    zero = np.zeros(256, np.float32)
    a = g.add_conv(0, materialise(rng.standard_normal((256, 256, 1, 1)) / 16, "bf16"), zero, act="relu")
    b = g.add_conv(a, materialise(rng.standard_normal((256, 256, 3, 3)) / 48, "bf16"), zero, pad=1)
    s = g.add_add(b, a, "relu")
    g.profile(warmup=5, reps=20)
    costs = g.costs()
    nhwc = {i: {r["rid"]: r["ns"] for r in costs["layers"][i]["routines"] if r["layout"] == N.NHWC}
            for i in (a, b, s)}
    add = next(iter(nhwc[s]))
    slow, fast = max(nhwc[a], key=nhwc[a].get), min(nhwc[a], key=nhwc[a].get)
    fused = set()
    for r in nhwc[b]:
        g.set_path([0, fast, r, add])
        if b not in g.plan_launches():
            fused.add(r)
    pairs = [(abs(nhwc[b][f] - nhwc[b][o] - 1300), f, o) for f in fused for o in nhwc[b]
             if o not in fused and nhwc[b][o] <= 0.9 * nhwc[b][f] and nhwc[b][f] <= nhwc[b][o] + 1600]
    assert pairs, "no pair of routines a little apart"
    _, f, o = min(pairs)
    print("with the addition", nhwc[b][f], "ns, without", nhwc[b][o], "ns; first layer", nhwc[a][slow], nhwc[a][fast])
    for l in costs["layers"][1:-1]:                # only these routines, as near ties
        for r in l["routines"]:
            r["ns"] = 10000 if (l["id"], r["rid"]) in {(a, slow), (a, fast), (b, f), (b, o), (s, add)} else -1
            r.pop("child", None)
    g.set_costs(costs)
    g.set_path([0, slow, f, add])
    launches = len(g.plan_launches())
    n = g.refine_in_path(tol_permille=100, max_alts=3, reps=15)
    assert g.path()[0] == [0, fast, f, add] and n == 1
    assert len(g.plan_launches()) <= launches
    g.close()


@pytest.mark.parametrize("name", ["resnet18", "mobilenetv2", "resnet50_bf16", "resnet50_f16",
                                  "resnet50_fused", "resnet50_proj", "mobilenetv2_fused", "vgg16_64px"])
def test_net_dp_and_fixed_paths_match_oracle(name):
    spec = {"resnet18": lambda: resnet18(1), "mobilenetv2": lambda: mobilenet_v2(1),
            "vgg16_64px": lambda: vgg16(2, "bf16", 64),
            "resnet50_bf16": lambda: resnet50(1, "bf16"),
            "resnet50_f16": lambda: resnet50(1, "f16"),
            "resnet50_fused": lambda: fuse_residual(resnet50(1, "bf16")),
            "resnet50_proj": lambda: fuse_projection(fuse_residual(resnet50(1, "bf16"))),
            "mobilenetv2_fused": lambda: fuse_residual(mobilenet_v2(1))}[name]()
    t = generate(spec)
    g = build_from_spec(spec, t)
    g.profile(warmup=2, reps=5)
    ref = oracle_out(spec, t)
    g.select("dprs")
    out, _ = run_out(g, spec, t)
    e = err(out, ref, spec["dtype"])
    print(f"{name} dprs err {e:.3e}", flush=True)
    assert e <= TOL[spec["dtype"]]
    costs = g.costs()
    tt, tup = blockwise(problem_from_costs(costs), [0, 1, 2])
    assert tuple(g.path()[0]) + (0,) == tup and g.path()[1] == tt
    for lay in ("NCHW", "NHWC", "NC8HW8"):
        for algo in ("igemm", "winograd", "direct"):
            g.select("fixed", lay, algo)
            out, _ = run_out(g, spec, t)
            e = err(out, ref, spec["dtype"])
            print(f"{name} fixed {lay}/{algo} err {e:.3e}", flush=True)
            assert e <= TOL[spec["dtype"]], (lay, algo)
    g.close()


def test_workspace_limited_selection_runs_within_the_limit():
    # memory-restricted tuning: with no routine workspace allowed, the
    # profiled DP path of a bs2 ResNet-18 (split-reduction tiles and the
    # three-kernel Winograd left out) uses none, and matches the oracle
    spec = fuse_projection(fuse_residual(resnet18(2, "bf16")))
    t = generate(spec)
    free = build_from_spec(spec, t)
    g = build_from_spec(spec, t, ws_limit=0)
    n_layers = len(spec["layers"]) + 1
    assert sum(len(g.routines(i)) for i in range(1, n_layers)) < sum(len(free.routines(i)) for i in range(1, n_layers))
    free.close()
    g.profile(warmup=2, reps=5)
    g.select("dprs")
    ids, _ = g.path()
    assert all(g.routines(i)[ids[i]]["ws_bytes"] == 0 for i in range(1, n_layers))
    out, _ = run_out(g, spec, t)
    e = err(out, oracle_out(spec, t), "bf16")
    print(f"resnet18 bs2 workspace-free dprs err {e:.3e}", flush=True)
    assert e <= TOL["bf16"]
    g.close()


@pytest.mark.parametrize("ws_limit", [0, None])
def test_workspace_limit_packs_the_intermediate_tensors(ws_limit):
    # six 12.8 MB maps in a chain: under a memory restriction two are alive at
    # a time; without one each gets bytes of its own (below 150 MiB in all)
    import torch
    from paper_2110_06037_amd import Graph
    rng = np.random.default_rng(3)
    g = Graph("bf16", 32, 64, 56, 56, device=0, layouts=["NHWC"], algos=["igemm"], ws_limit=ws_limit)
    last = 0
    for _ in range(5):
        last = g.add_conv(last, materialise(rng.standard_normal((64, 64, 1, 1)) / 8, "bf16"), np.zeros(64, np.float32),
                          act="relu")
    size = 32 * 64 * 56 * 56 * 2
    ids = [0] + [next(r["id"] for r in g.routines(i) if r["ws_bytes"] == 0) for i in range(1, last + 1)]
    before = torch.cuda.mem_get_info()[0]
    g.set_path(ids)
    held = before - torch.cuda.mem_get_info()[0]
    maps = 2 if ws_limit == 0 else 6           # the converted input and five outputs
    assert abs(held - maps * size) < size // 2
    g.close()


def test_resnet50_bs32_dp_path_sampled_images():
    # the benchmark's configuration: full batch on the GPU, images 0 and 1
    # through the oracle (images are independent)
    spec = resnet50(32, "bf16")
    t = generate(spec)
    g = build_from_spec(spec, t)
    g.profile(warmup=2, reps=5)
    g.select("dprs")
    out, _ = run_out(g, spec, t)
    ref = oracle_out(spec, t, images=2)
    e = err(out[:2], ref, "bf16")
    print(f"resnet50 bs32 dprs images 0-1 err {e:.3e}", flush=True)
    assert e <= TOL["bf16"]
    assert np.all(np.isfinite(out))
    g.close()


@pytest.mark.parametrize("si", range(len(CONV_SWEEP_SHAPES)))
def test_conv_sweep_full_size_sampled(si):
    # full-size layer (batch 32, fp16): every routine checked on 3000 sampled outputs
    c, hw = CONV_SWEEP_SHAPES[si]
    spec = conv_sweep(c, hw)
    t = generate(spec)
    g = build_from_spec(spec, t)
    xd = to_dev(t["x"], "f16")
    x64 = to_f64(t["x"], "f16")
    w64 = to_f64(t["w"][0], "f16")
    b64 = t["b"][0].astype(np.float64)
    rng = np.random.default_rng(si)
    idx = np.stack([rng.integers(0, 32, 3000), rng.integers(0, c, 3000),
                    rng.integers(0, hw, 3000), rng.integers(0, hw, 3000)], axis=1)
    ref = O.round_to(O.conv2d_points(x64, w64, b64, idx, 1, 1, 1, "none"), "f16")
    import torch
    for rt in g.routines(1):
        g.set_path([0, rt["id"]])
        y = g.run(xd)
        torch.cuda.synchronize()
        y = from_dev(y, "f16")
        got = y[idx[:, 0], idx[:, 1], idx[:, 2], idx[:, 3]]
        e = err(got, ref, "f16")
        print(f"sweep c{c} {rt['name']} err {e:.2e}", flush=True)
        assert e <= TOL["f16"], rt["name"]
    g.close()


def test_hip_graph_replays_match_eager():
    import torch
    spec = resnet18(1)
    t = generate(spec)
    g = build_from_spec(spec, t)
    g.select("fixed", "NHWC", "igemm")
    eager, xd = run_out(g, spec, t)
    g.set_option(N.OPT_HIPGRAPH, 1)
    for rep in range(4):
        y = g.run(xd)
        torch.cuda.synchronize()
        got = from_dev(y, "bf16").reshape(1, -1)
        assert np.array_equal(got, eager), rep
        junk = torch.randn(1 << 20, device="cuda").sum()   # eager work between replays
        torch.cuda.synchronize()
    g.close()


def _images_out(g, spec, t, images):
    import torch
    xd = to_dev(t["x"], spec["dtype"])
    y = g.run(xd)
    torch.cuda.synchronize()
    out = from_dev(y, spec["dtype"]).reshape(spec["batch"], -1)
    d = decoded(t, spec["dtype"])
    d["x"] = d["x"][images]
    ref = O.forward(with_batch(spec, len(images)), d, storage="dtype")[-1]
    return out, out[images], ref.reshape(len(images), -1)


FULL_BATCH = {
    # name: (spec factory, images through the oracle: first, middle, last)
    "resnet50_bs32_bf16_proj": (lambda: fuse_projection(fuse_residual(resnet50(32, "bf16"))), [0, 13, 31]),
    "resnet50_bs32_f16_proj": (lambda: fuse_projection(fuse_residual(resnet50(32, "f16"))), [1, 19, 30]),
    "resnet50_bs32_bf16_fused": (lambda: fuse_residual(resnet50(32, "bf16")), [0, 13, 31]),
    "resnet50_bs32_f16_fused": (lambda: fuse_residual(resnet50(32, "f16")), [0, 17, 31]),
    "resnet50_bs32_f16": (lambda: resnet50(32, "f16"), [2, 31]),
    "mobilenetv2_bs8_fused": (lambda: fuse_residual(mobilenet_v2(8)), [0, 3, 7]),
    "mobilenetv2_bs8": (lambda: mobilenet_v2(8), [1, 6]),
    "vgg16_bs32_224": (lambda: vgg16(32, "bf16"), [0, 31]),
}


@pytest.mark.parametrize("name", list(FULL_BATCH))
def test_full_batch_paths_on_images_across_the_batch(name):
    # the benchmark's configurations at their full batch: the DPRS path and
    # the path integrated profiling keeps (the one bench.py times), checked
    # on images at the start, middle and end of the batch, so that tiles far
    # from the first of every persistent workgroup are compared too
    make, images = FULL_BATCH[name]
    spec = make()
    t = generate(spec)
    g = build_from_spec(spec, t)
    g.profile(warmup=2, reps=5)
    g.select("dprs")
    out, got, ref = _images_out(g, spec, t, images)
    e = err(got, ref, spec["dtype"])
    print(f"{name} dprs images {images} err {e:.3e}", flush=True)
    assert e <= TOL[spec["dtype"]]
    assert np.all(np.isfinite(out))
    dprs_ids = g.path()[0]
    g.profile_integrated(warmup=2, reps=3)
    if g.path()[0] != dprs_ids:
        out, got, ref2 = _images_out(g, spec, t, images)
        e = err(got, ref, spec["dtype"])
        print(f"{name} selected path images {images} err {e:.3e}", flush=True)
        assert e <= TOL[spec["dtype"]]
        assert np.all(np.isfinite(out))
    g.close()


def _rotating_layout_path(g):
    # a routine of layout (i mod 3) on layer i where one exists (implicit
    # GEMM first): a converter on almost every edge
    ids = [0]
    for i in range(1, g.num_layers()):
        rts = g.routines(i)
        want = [r for r in rts if r["layout"] == i % 3] or rts
        ids.append(min(want, key=lambda r: (r["algo"] != 1, r["id"]))["id"])
    return ids


def test_run_timed_equals_run_on_a_mixed_layout_path():
    # sn_run_timed repeats every layer's converters and routine; a converter's
    # source must outlive the layer's routine, so the repeated run gives the
    # same bits as sn_run on a path that switches layout on every edge
    import torch
    spec = resnet18(1)
    t = generate(spec)
    g = build_from_spec(spec, t)
    ids = _rotating_layout_path(g)
    g.set_path(ids)
    layouts = [g.routines(i)[ids[i]]["layout"] for i in range(len(ids))]
    assert len(set(layouts[1:])) == 3
    out, xd = run_out(g, spec, t)
    assert err(out, oracle_out(spec, t), "bf16") <= TOL["bf16"]
    for reps in (3, 1):
        y, ms = g.run_timed(xd, reps=reps)
        torch.cuda.synchronize()
        assert np.array_equal(from_dev(y, "bf16").reshape(1, -1), out), reps
        assert all(m > 0 for m in ms[1:])
    g.close()


def odd_channel_net():
    """Channel counts that are not multiples of 8 on every layer: NC8HW8
    stores them padded."""
    L = [
        {"type": "conv", "in": [0], "k": 12, "r": 3, "s": 3, "stride": 1, "pad": 1, "groups": 1, "act": "relu"},
        {"type": "conv", "in": [1], "k": 12, "r": 3, "s": 3, "stride": 2, "pad": 1, "groups": 12, "act": "relu6"},
        {"type": "conv", "in": [2], "k": 20, "r": 1, "s": 1, "stride": 1, "pad": 0, "groups": 1, "act": "none"},
        {"type": "maxpool", "in": [3], "k": 3, "stride": 1, "pad": 1},
        {"type": "conv", "in": [4], "k": 20, "r": 3, "s": 3, "stride": 1, "pad": 1, "groups": 1, "act": "none"},
        {"type": "add", "in": [5, 3], "act": "relu"},
        # a 1x1 convolution with a folded residual input (layer 4)
        {"type": "conv", "in": [6, 4], "k": 20, "r": 1, "s": 1, "stride": 1, "pad": 0, "groups": 1, "act": "relu"},
        {"type": "gap", "in": [7]},
        {"type": "fc", "in": [8], "k": 10},
    ]
    return {"name": "odd_channels", "dtype": "bf16", "batch": 3, "in_chw": [3, 13, 11],
            "input_dist": "uniform", "seed": 5, "layers": L,
            "layouts": ["NCHW", "NHWC", "NC8HW8"], "algos": ["direct", "igemm", "winograd"]}


@pytest.mark.parametrize("algo", ["igemm", "direct", "winograd"])
def test_nc8hw8_stored_outputs_keep_padded_channels_zero(algo):
    # every layer's output as its NC8HW8 routine stored it: the channels
    # padded up to a multiple of 8 hold exact zeros, and the real channels
    # hold the oracle's layer output
    import torch
    spec = odd_channel_net()
    t = generate(spec)
    g = build_from_spec(spec, t)
    g.set_option(N.OPT_KEEP, 1)
    g.select("fixed", "NC8HW8", algo)
    xd = to_dev(t["x"], "bf16")
    y = g.run(xd)
    torch.cuda.synchronize()
    refs = O.forward(spec, decoded(t, "bf16"), storage="dtype", keep=True)
    for i in range(1, g.num_layers()):
        n, c, h, w = g.layer_shape(i)
        try:
            buf, lay = g.layer_output(i)
        except N.SNError as e:
            assert i == g.num_layers() - 1 and e.code == -4, e   # stored into the user's output
            continue
        torch.cuda.synchronize()
        assert lay == N.NC8HW8
        c8 = (c + 7) // 8 * 8
        bits = buf.cpu().numpy().view(np.uint16)
        assert bits.size == n * c8 * h * w, (i, bits.size)
        blk = bits.reshape(n, c8 // 8, h, w, 8).transpose(0, 1, 4, 2, 3).reshape(n, c8, h, w)
        assert not np.any(blk[:, c:]), f"layer {i}: padded channels hold non-zero bits"
        got = to_f64(blk[:, :c], "bf16")
        e = err(got, refs[i].reshape(n, c, h, w), "bf16")
        print(f"odd-channel net {algo} layer {i} err {e:.2e}", flush=True)
        assert e <= TOL["bf16"], i
    out = from_dev(y, "bf16").reshape(3, -1)
    assert err(out, refs[-1].reshape(3, -1), "bf16") <= TOL["bf16"]
    g.close()


def test_plan_launch_list_matches_the_routines():
    # sn_plan_launches lists a run's kernel launches by layer without
    # launching anything: every layer appears in order, a Winograd layer
    # with its three kernels (input transform, tile GEMMs, output transform),
    # converters before the layer they feed; the next run is unaffected
    import torch
    spec = resnet18(1)
    t = generate(spec)
    g = build_from_spec(spec, t)
    g.select("fixed", "NHWC", "winograd")
    out0, xd = run_out(g, spec, t)
    ids = g.path()[0]
    lay = g.plan_launches()
    assert lay == sorted(lay) and set(lay) == set(range(1, g.num_layers()))
    for i in range(1, g.num_layers()):
        rt = g.routines(i)[ids[i]]
        n = lay.count(i)
        conv = 1 if i == 1 else 0          # the input's NCHW -> NHWC converter feeds layer 1
        if rt["algo"] == N.WINOGRAD:
            assert n == 3 + conv, (i, rt["name"], n)
        elif i == 1:
            assert n == 2, (i, rt["name"], n)
    out1, _ = run_out(g, spec, t)
    assert np.array_equal(out0, out1)
    g.close()


@pytest.mark.parametrize("hw", [20, 247, 250])
def test_adapts_making_one_conversion_share_its_result(hw):
    # x enters the first convolution and, as the residual, the last one, both
    # in NHWC: one converter serves both.  At 247 x 247 the converted copy,
    # alive beside the two 256-channel maps, takes the plan past the 64 MiB of
    # sn_run_noalloc, which there runs a layout that converts per edge; at 250
    # x 250 that one still fits (61.0 MiB).
    import torch
    from paper_2110_06037_amd import Graph
    rng = np.random.default_rng(7)

    def wts(k, c):
        return materialise(rng.standard_normal((k, c, 1, 1)) * np.sqrt(2 / c), "bf16")
    w = [wts(256, 64), wts(256, 256), wts(64, 256)]
    b = [np.zeros(k, np.float32) for k in (256, 256, 64)]
    g = Graph("bf16", 1, 64, hw, hw, layouts=["NHWC"], algos=["igemm"])
    a = g.add_conv(0, w[0], b[0], act="relu")
    a = g.add_conv(a, w[1], b[1], act="relu")
    g.add_conv(a, w[2], b[2], act="relu", residual=0)
    g.select("fixed", "NHWC", "igemm")
    assert g.plan_launches() == [1, 1, 2, 3, 3]
    x = materialise(rng.standard_normal((1, 64, hw, hw)), "bf16")
    xd = to_dev(x, "bf16")
    out = g.run(xd)
    f = [to_f64(v, "bf16").reshape(v.shape[:2]) for v in w]
    px = to_f64(x, "bf16").reshape(64, -1)[:, ::97]
    h = px
    for m in f[:2]:
        h = np.maximum(m @ h, 0)
    ref = np.maximum(f[2] @ h + px, 0)
    assert err(from_dev(out, "bf16").reshape(64, -1)[:, ::97], ref, "bf16") <= TOL["bf16"]
    again, _ = g.run_timed(xd, reps=3)
    out2 = torch.empty_like(out)
    g.run_noalloc(xd, out2)
    torch.cuda.synchronize()
    assert torch.equal(out, again) and torch.equal(out, out2)
    g.close()


def test_noalloc_run_without_the_fused_launches():
    # 47 images of 3 x 56 x 56 through a stem, two 3x3 layers and an addition,
    # maps of 18.9 MB: with the addition in its convolution's launch four are
    # alive at once (72 MiB), layer by layer three (54 MiB), so sn_run_noalloc
    # runs the layers one by one, the stem behind its converter, to the same bits
    import torch
    from paper_2110_06037_amd import Graph
    rng = np.random.default_rng(9)
    n, k, hw = 47, 64, 56
    g = Graph("bf16", n, 3, hw, hw, device=0, layouts=["NHWC"], algos=["igemm"])

    def wts(c):
        return materialise(rng.standard_normal((k, c, 3, 3)) / np.sqrt(4.5 * c), "bf16")
    b = rng.uniform(-0.1, 0.1, k).astype(np.float32)
    ws = [wts(3), wts(k), wts(k)]
    stem = g.add_conv(0, ws[0], b, pad=1, act="relu")
    c1 = g.add_conv(stem, ws[1], b, pad=1, act="relu")
    c2 = g.add_conv(c1, ws[2], b, pad=1)
    a = g.add_add(c2, stem, "relu")

    def fewest(layer, ids):
        best = None
        for r in g.routines(layer):
            if r["ws_bytes"]:
                continue
            g.set_path(ids[:layer] + [r["id"]] + ids[layer + 1:])
            m = len(g.plan_launches())
            if best is None or m < best[0]:
                best = (m, r["id"])
        return ids[:layer] + [best[1]] + ids[layer + 1:]
    plain = [next(r["id"] for r in g.routines(i) if r["ws_bytes"] == 0) for i in range(1, a + 1)]
    ids = fewest(c2, fewest(stem, [0] + plain))
    g.set_path(ids)
    # the stem without its converter, the addition in c2's launch, the output's converter
    assert g.plan_launches() == [stem, c1, a, a]
    x = materialise(rng.uniform(-1, 1, (n, 3, hw, hw)), "bf16")
    xd = to_dev(x, "bf16")
    out = g.run(xd)
    d = [to_f64(w, "bf16") for w in ws]
    x1, b64 = to_f64(x[:1], "bf16"), b.astype(np.float64)
    s0 = O.round_to(O.conv2d(x1, d[0], b64, 1, 1, 1, "relu"), "bf16")
    h = O.round_to(O.conv2d(s0, d[1], b64, 1, 1, 1, "relu"), "bf16")
    h = O.round_to(O.conv2d(h, d[2], b64, 1, 1), "bf16")
    assert err(from_dev(out, "bf16")[:1], O.round_to(O.add(h, s0, "relu"), "bf16"), "bf16") <= TOL["bf16"]
    out2 = torch.zeros_like(out)
    g.run_noalloc(xd, out2)
    torch.cuda.synchronize()
    assert torch.equal(out, out2)
    g.close()


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
# (C, K, H, W, R, act, addition's operand order): ragged pixel and channel
# tiles; K % 8 != 0 (element stores); every patch tile applies at 64 channels
@pytest.mark.parametrize("case", [(64, 64, 14, 14, 3, "relu", 0), (64, 72, 28, 28, 3, "none", 1),
                                  (32, 20, 9, 7, 3, "relu6", 0), (24, 40, 5, 6, 1, "relu", 1),
                                  (64, 64, 56, 56, 3, "relu", 0)])
def test_addition_in_its_convolutions_launch(dtype, case):
    # a convolution read by one addition alone, in its schema, without an
    # activation: one launch, with the bits of the two (a timed run makes both)
    import torch
    from paper_2110_06037_amd import Graph
    c, k, h, w, r, act, order = case
    n = 2
    rng = np.random.default_rng(11)
    wt = materialise(rng.standard_normal((k, c, r, r)) * np.sqrt(2 / (c * r * r)), dtype)
    b = rng.uniform(-0.1, 0.1, k).astype(np.float32)
    x = materialise(rng.uniform(-1, 1, (n, c, h, w)), dtype)
    x2 = materialise(rng.uniform(-1, 1, (n, k, h, w)), dtype)
    x2.reshape(-1)[3] = materialise(np.array([np.inf]), dtype)[0]
    ref = O.round_to(O.conv2d(to_f64(x, dtype), to_f64(wt, dtype), b.astype(np.float64), 1, r // 2), dtype)
    ref = O.round_to(O.add(ref, to_f64(x2, dtype), act), dtype).reshape(-1)
    fin = np.isfinite(ref)
    g = Graph(dtype, n, c, h, w, device=0, algos=["igemm"])
    i2 = g.add_input(k, h, w)
    cv = g.add_conv(0, wt, b, pad=r // 2)
    a = g.add_add(*((cv, i2) if order else (i2, cv)), act)
    adds = {rt["layout"]: rt["id"] for rt in g.routines(a)}
    xs = [to_dev(x, dtype), to_dev(x2, dtype)]
    fused = set()
    for rt in g.routines(cv):
        if rt["algo"] != N.IGEMM:
            continue
        g.set_path([0, 0, rt["id"], adds[rt["layout"]]])
        lay = g.plan_launches()
        if cv in lay and lay.count(cv) > (1 if rt["layout"] else 0):
            continue                                             # two launches
        fused.add(rt["param"])
        out = g.run_mimo(xs, output_layers=[a])[0]
        got = from_dev(out, dtype).reshape(-1)
        assert err(got[fin], ref[fin], dtype) <= TOL[dtype], rt["name"]
        assert not np.isfinite(got[~fin]).any() if act != "relu6" else (got[~fin] == 6).all(), rt["name"]
        g.set_option(N.OPT_KEEP, 1)                              # both layers' outputs kept: two launches
        assert g.plan_launches().count(cv) > lay.count(cv)
        two = g.run_mimo(xs, output_layers=[a])[0]
        torch.cuda.synchronize()
        assert torch.equal(out, two), rt["name"]
        g.set_option(N.OPT_KEEP, 0)
    assert fused if dtype == "f32" else {p for p in fused if p >= 106}
    if dtype != "f32" and r == 3 and k % 8 == 0 and c == 64:
        assert {p for p in fused if p < 106}                     # patch tiles too
    g.close()


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("case", [  # (N, C, H, W, K, R, stride, pad)
    (2, 3, 40, 46, 64, 7, 2, 3), (1, 3, 225, 224, 24, 7, 2, 3), (3, 4, 17, 22, 24, 3, 2, 1), (2, 2, 9, 16, 72, 3, 1, 1),
    (2, 3, 21, 18, 8, 5, 2, 2), (1, 3, 12, 14, 16, 3, 1, 0), (5, 3, 1, 2, 8, 3, 1, 1), (2, 3, 8, 9, 8, 3, 1, 1)])
def test_images_read_from_nchw_by_the_small_channel_kernel(dtype, case):
    """The small-channel kernel reads the caller's planes itself (even widths):
    the bits of the plan that converts them first, with one launch less; on
    images that are only 2-byte aligned the converter runs."""
    import torch
    from paper_2110_06037_amd import Graph
    from workloads import random_tensor
    n, c, h, w, k, r, st, pad = case
    x = random_tensor((n, c, h, w), dtype, seed=71)
    wt = random_tensor((k, c, r, r), dtype, seed=72, dist="normal", scale=np.sqrt(2 / (c * r * r)))
    b = random_tensor((k,), "f32", seed=73, scale=0.1)
    xd = to_dev(x, dtype)
    off = torch.empty(xd.numel() + 1, dtype=xd.dtype, device="cuda")[1:].view(xd.shape).copy_(xd)
    outs, launches = [], []
    for keep in (1, 0):
        g = Graph(dtype, n, c, h, w, device=0, layouts=["NCHW", "NHWC"], algos=["igemm"])
        g.set_option(N.OPT_KEEP, keep)
        g.add_conv(0, wt, b, st, pad, act="relu")
        g.add_maxpool(1, 2, 2, 0) if min(h, w) > 4 else g.add_add(1, 1)
        second = [q["id"] for q in g.routines(2) if q["layout"] == 1][0]
        ids = [q["id"] for q in g.routines(1) if q["layout"] == 1]
        assert ids
        for rid in ids:
            g.set_path([0, rid, second])
            outs.append([g.run(t).cpu() for t in (xd, off)])
            launches.append(len(g.plan_launches()))
        g.close()
    m = len(ids)
    for a, z in zip(outs[:m], outs[m:]):
        assert all(torch.equal(a[0], t) for t in (a[1], z[0], z[1]))
    fewer = [a - z for a, z in zip(launches[:m], launches[m:])]
    assert set(fewer) <= {0, 1} and (1 in fewer) == (w % 2 == 0)
