"""GPU tests of batching: mixed-distance groups in one call, HIP-graph capture and replay, and the launch
variants the autotuner chooses among. Every variant must give results identical to a plain decode of each
group alone, and a mixed call is also checked against the FP64 oracle."""
import sys

import numpy as np
import pytest

from oracle import blockbp
from paper_2402_04834_amd import workload

pytestmark = pytest.mark.gpu

KEYS = ("loglik", "delta", "iters", "coset", "correction")


def _say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def dev():
    import torch
    import paper_2402_04834_amd as bbp
    bbp._lib.lib()
    return torch.device("cuda:0")


def _np(out):
    return {k: out[k].cpu().numpy() for k in KEYS}


def _alone(dev, d, p, syn, opts):
    import torch
    import paper_2402_04834_amd as bbp
    out = bbp.decode_device(d, p, torch.from_numpy(syn).to(dev), opts)
    torch.cuda.synchronize()
    return _np(out)


def _same(a, b, what):
    for k in KEYS:
        np.testing.assert_array_equal(a[k], b[k], err_msg=f"{what}: {k}")


MIX = [(5, 0.10, 7), (7, 0.08, 5), (9, 0.12, 3), (11, 0.10, 2), (17, 0.10, 3)]


def _mix_inputs():
    return [(d, p, workload.make_batch(d, p, b, workload="mixed", p_index=d)[1]) for d, p, b in MIX]


@pytest.mark.parametrize("precision", [0, 1])
def test_mixed_groups_equal_separate_decodes(dev, precision):
    # FP32, and precision mode 1 (BF16 matrix-core contractions): batching never changes a result
    import torch
    import paper_2402_04834_amd as bbp
    opts = bbp.default_opts(block=6, chi=32, max_iter=12, precision=precision)
    inputs = _mix_inputs()
    _say("[mixed] groups", [(d, p, s.shape[0]) for d, p, s in inputs], "precision", precision)
    outs, _, _ = bbp.decode_groups([(d, p, torch.from_numpy(s).to(dev)) for d, p, s in inputs], opts)
    torch.cuda.synchronize()
    for (d, p, s), o in zip(inputs, outs):
        _same(_np(o), _alone(dev, d, p, s, opts), f"d={d}")


def test_mixed_groups_against_oracle(dev):
    import torch
    import paper_2402_04834_amd as bbp
    opts = bbp.default_opts(block=6, chi=32, max_iter=4, fixed_iters=1)
    inputs = [(5, 0.10, workload.make_batch(5, 0.10, 4, workload="mixed", p_index=50)[1]),
              (7, 0.09, workload.make_batch(7, 0.09, 3, workload="mixed", p_index=70)[1])]
    _say("[mixed oracle] d=5 x4, d=7 x3, fixed 4 iterations")
    outs, _, _ = bbp.decode_groups([(d, p, torch.from_numpy(s).to(dev)) for d, p, s in inputs], opts)
    torch.cuda.synchronize()
    for (d, p, s), o in zip(inputs, outs):
        ref = blockbp.decode(d, p, s, block=(6, 6), chi=32, max_iter=4, fixed_iters=True)
        got = o["loglik"].cpu().numpy()
        np.testing.assert_allclose(got, ref["loglik"], atol=2e-4 + 2e-6 * np.abs(ref["loglik"]).max())
        np.testing.assert_array_equal(o["coset"].cpu().numpy(), ref["coset"])


def test_graph_replays_match_eager(dev):
    import torch
    import paper_2402_04834_amd as bbp
    d, p = 9, 0.10
    _, syn = workload.make_batch(d, p, 16, workload="mixed", p_index=90)
    eager_opts = bbp.default_opts(block=6, chi=32, max_iter=10)
    ref = _alone(dev, d, p, syn, eager_opts)
    graph_opts = bbp.default_opts(block=6, chi=32, max_iter=10, graph=1)
    st = torch.cuda.Stream(dev)
    syn_dev = torch.from_numpy(syn).to(dev)
    ws = torch.empty(bbp.workspace_size(d, 16, graph_opts), dtype=torch.uint8, device=dev)
    other = torch.from_numpy(workload.make_batch(d, p, 8, workload="mixed", p_index=91)[1]).to(dev)
    out = None
    for rep in range(4):
        _say(f"[graph] {'capture' if rep == 0 else 'replay'} {rep}")
        with torch.cuda.stream(st):
            out = bbp.decode_device(d, p, syn_dev, graph_opts, workspace=ws, stream=st, out=out)
        st.synchronize()
        _same(_np(out), ref, f"replay {rep}")
        # eager work of the program between replays, on the default stream
        bbp.decode_device(d, p, other, eager_opts)
        torch.cuda.synchronize()


def test_graph_capture_of_multi_stream_rounds(dev):
    """A decode whose rounds spread over 4 streams (fork / join events) captures into one graph; its replays
    equal the eager decode bitwise."""
    import torch
    import paper_2402_04834_amd as bbp
    d, p = 9, 0.10
    _, syn = workload.make_batch(d, p, 16, workload="mixed", p_index=95)
    eager_opts = bbp.default_opts(block=6, chi=32, max_iter=10)
    bbp.set_tuning(d, eager_opts, 1, 4)
    ref = _alone(dev, d, p, syn, eager_opts)
    graph_opts = bbp.default_opts(block=6, chi=32, max_iter=10, graph=1)
    st = torch.cuda.Stream(dev)
    syn_dev = torch.from_numpy(syn).to(dev)
    ws = torch.empty(bbp.workspace_size(d, 16, graph_opts), dtype=torch.uint8, device=dev)
    out = None
    for rep in range(3):
        _say(f"[graph 4 streams] {'capture' if rep == 0 else 'replay'} {rep}")
        with torch.cuda.stream(st):
            out = bbp.decode_device(d, p, syn_dev, graph_opts, workspace=ws, stream=st, out=out)
        st.synchronize()
        _same(_np(out), ref, f"replay {rep}")
    bbp.set_tuning(d, eager_opts, 0, 1)


def test_launch_variants_give_identical_results(dev):
    import torch
    import paper_2402_04834_amd as bbp
    d, p = 11, 0.10
    _, syn = workload.make_batch(d, p, 12, workload="mixed", p_index=110)
    opts = bbp.default_opts(block=6, chi=32, max_iter=15)
    bbp.set_tuning(d, opts, 0, 1)
    ref = _alone(dev, d, p, syn, opts)
    for order in (0, 1):
        for streams in (1, 2, 4):
            _say(f"[variant] order={order} streams={streams}")
            bbp.set_tuning(d, opts, order, streams)
            _same(_alone(dev, d, p, syn, opts), ref, f"order {order} streams {streams}")
    best = bbp.autotune(d, p, torch.from_numpy(syn).to(dev), opts)
    torch.cuda.synchronize()
    assert best.order in (0, 1) and best.streams in (1, 2, 4) and best.ms > 0
    _same(_alone(dev, d, p, syn, opts), ref, "autotuned")
    bbp.set_tuning(d, opts, 0, 1)


def test_host_api_mixed_networks_in_input_order(dev):
    import paper_2402_04834_amd as bbp
    opts = bbp.default_opts(block=6, chi=32, max_iter=8)
    items = []
    for d, p in ((5, 0.1), (7, 0.1), (5, 0.1), (9, 0.08), (7, 0.1)):
        _, s = workload.make_batch(d, p, 1, workload="mixed", p_index=100 + d, start=len(items))
        items.append((d, p, s[0]))
    _say("[host mixed] 5 networks of d 5, 7, 9")
    nets = [bbp.build_network(d, p, s) for d, p, s in items]
    got = bbp.blockbp_decode(nets, opts)
    nmax = got["correction"].shape[1]
    assert nmax == 9 * 9 + 8 * 8
    for i, (d, p, s) in enumerate(items):
        ref = _alone(dev, d, p, s[None, :], opts)
        n = d * d + (d - 1) * (d - 1)
        np.testing.assert_array_equal(got["loglik"][i], ref["loglik"][0])
        np.testing.assert_array_equal(got["iters"][i], ref["iters"][0])
        assert got["coset"][i] == ref["coset"][0]
        np.testing.assert_array_equal(got["correction"][i, :n], ref["correction"][0])
        assert np.all(got["correction"][i, n:] == 0)


def _mixed_workload(count):
    """The mixed-distance workload: per syndrome d uniform over {9, 13, 17, 21} and p uniform over
    [0.05, 0.15]; chi 16 for d <= 13 and 32 above. Returns {d: (indices, p array, syndromes)}."""
    items = workload.mixed_batch(count)
    groups = {}
    for i, (d, p, _, s) in enumerate(items):
        groups.setdefault(d, ([], [], []))
        groups[d][0].append(i)
        groups[d][1].append(p)
        groups[d][2].append(s)
    return {d: (np.array(ix), np.array(ps), np.stack(ss)) for d, (ix, ps, ss) in sorted(groups.items())}


def test_mixed_distance_workload_one_graph(dev):
    import torch
    import paper_2402_04834_amd as bbp
    mix = _mixed_workload(8192)
    _say("[mixed workload] 8192 syndromes:", {d: len(v[0]) for d, v in mix.items()})
    opts = bbp.default_opts(block=6, chi=32, max_iter=20, graph=1)
    chi_of = {9: 16, 13: 16, 17: 32, 21: 32}
    groups = [(d, torch.from_numpy(ps).to(dev), torch.from_numpy(ss).to(dev), chi_of[d])
              for d, (ix, ps, ss) in mix.items()]
    st = torch.cuda.Stream(dev)
    with torch.cuda.stream(st):
        outs, ws, _ = bbp.decode_groups(groups, opts, stream=st)
    st.synchronize()
    # each group decoded alone (eager) gives identical results
    eager = bbp.default_opts(block=6, chi=32, max_iter=20)
    for (d, p_t, s_t, chi), o in zip(groups, outs):
        _say(f"[mixed workload] d={d} alone")
        alone, _, _ = bbp.decode_groups([(d, p_t, s_t, chi)], eager)
        torch.cuda.synchronize()
        _same(_np(o), _np(alone[0]), f"d={d}")
        assert np.all(o["coset"].cpu().numpy() < 4)
    # oracle parity on the committed fixture: the first 64 syndromes of every distance, each at its own p
    # (tests/golden/mixed_8192_first64_per_d.json, written by make_oracle_fixtures.py from oracle/ only)
    import json
    import os
    path = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "mixed_8192_first64_per_d.json")
    fx = json.load(open(path))
    assert fx["meta"]["count"] == 8192 and fx["meta"]["max_iter"] == 20
    per_d = {}
    for r in fx["records"]:
        d = r["d"]
        ix, ps, _ = mix[d]
        j = int(np.nonzero(ix == r["index"])[0][0])
        assert abs(ps[j] - r["p"]) < 1e-15 and r["chi"] == chi_of[d]
        per_d.setdefault(d, []).append((j, r))
    for d, recs in sorted(per_d.items()):
        o = _np(outs[list(mix).index(d)])
        j = np.array([jj for jj, _ in recs])
        ref_ll = np.array([r["loglik"] for _, r in recs])
        ref_dl = np.array([r["delta"] for _, r in recs])
        ref_it = np.array([r["iters"] for _, r in recs])
        ref_cs = np.array([r["coset"] for _, r in recs])
        it, ll = o["iters"][j], o["loglik"][j]
        near = np.abs(np.log(np.maximum(ref_dl, 1e-30) / 1e-4)) < 0.05
        assert np.all((it == ref_it) | near), f"d={d}"
        same = (it == ref_it) & np.isfinite(ref_ll)
        np.testing.assert_array_less(np.abs(ll[same] - ref_ll[same]), 2e-4 + 2e-6 * np.abs(ref_ll[same]))
        bad = o["coset"][j] != ref_cs
        for i in np.nonzero(bad)[0]:   # only ties within the FP32 error may differ
            trusted = ref_dl[i] < 1e-2
            cand = np.where(trusted, ref_ll[i], -np.inf) if trusted.any() else -ref_dl[i]
            srt = np.sort(cand)[::-1]
            assert srt[0] - srt[1] < 1e-3, (d, i, ref_ll[i], ref_dl[i])
        _say(f"[mixed workload] d={d}: {len(recs)} oracle records, decisions equal {int((~bad).sum())}, "
             f"max |dlnZ| {np.abs(ll[same] - ref_ll[same]).max():.2e}")

def test_concurrent_multistream_decodes_match_serial(dev):
    """Two host threads decoding at once with the four-stream launch variant (which shares the device's
    auxiliary streams and events), eagerly and through captured graphs, each on its own stream: every result
    is bitwise the serial decode's."""
    import threading
    import torch
    import paper_2402_04834_amd as bbp
    d, p = 9, 0.10
    opts = bbp.default_opts(block=6, chi=32, max_iter=20)
    gopts = bbp.default_opts(block=6, chi=32, max_iter=20, graph=1)
    bbp.set_tuning(d, opts, 1, 4)
    try:
        syn = [torch.from_numpy(workload.make_batch(d, p, 48, workload="mixed", p_index=120 + k)[1]).to(dev)
               for k in range(2)]
        ref = [_np(bbp.decode_device(d, p, s, opts)) for s in syn]
        torch.cuda.synchronize()
        errors, results = [], [[], []]

        def worker(k):
            try:
                st = torch.cuda.Stream(dev)
                ws = torch.empty(bbp.workspace_size(d, 48, opts), dtype=torch.uint8, device=dev)
                out = None
                for rep in range(6):
                    o = gopts if rep % 2 else opts
                    out = bbp.decode_device(d, p, syn[k], o, workspace=ws, stream=st, out=out)
                    st.synchronize()
                    results[k].append(_np(out))
            except Exception as e:   # reported by the main thread
                errors.append(e)

        _say("[concurrent] two threads, 4-stream variant, eager and graph")
        th = [threading.Thread(target=worker, args=(k,)) for k in range(2)]
        for t in th:
            t.start()
        for t in th:
            t.join()
        assert not errors, errors
        for k in range(2):
            assert len(results[k]) == 6
            for r in results[k]:
                _same(r, ref[k], f"thread {k}")
    finally:
        bbp.set_tuning(d, opts, 0, 1)


def test_strided_inputs_on_a_busy_side_stream(dev):
    """Syndromes, rates and start messages that are not contiguous are copied on the stream that decodes them: the
    current stream is kept busy, so a copy made there would not have run when the decode starts, and its memory is
    handed out again as soon as the call returns."""
    import torch
    import paper_2402_04834_amd as bbp
    d, b = 9, 24
    opts = bbp.default_opts(block=6, chi=32, max_iter=8)
    _, syn = workload.make_batch(d, 0.1, 2 * b, workload="test", p_index=77)
    s = torch.from_numpy(np.ascontiguousarray(syn)).to(dev)
    ps = torch.linspace(0.05, 0.15, 2 * b, dtype=torch.float64, device=dev)
    M = bbp.plan_query(d, opts).num_messages
    init = torch.rand((2 * b, 4, M, 64), generator=torch.Generator().manual_seed(5)).to(dev) + 0.1
    cut = [x[::2] for x in (s, ps, init)]
    assert not any(x.is_contiguous() for x in cut)
    whole = [x.contiguous() for x in cut]
    ref_one = _np(bbp.decode_device(d, 0.1, whole[0], opts))
    ref_all, _, _ = bbp.decode_groups([(d, whole[1], whole[0], 0, whole[2])], opts)
    torch.cuda.synchronize()
    st = torch.cuda.Stream(dev)
    _say("[strided] side stream, current stream busy")
    for _ in range(3):
        ws = torch.empty(bbp.workspace_size(d, b, opts), dtype=torch.uint8, device=dev)
        torch.cuda._sleep(20_000_000)
        one = bbp.decode_device(d, 0.1, cut[0], opts, workspace=ws, stream=st)
        torch.cuda._sleep(20_000_000)
        many, _, _ = bbp.decode_groups([(d, cut[1], cut[0], 0, cut[2])], opts, stream=st)
        junk = [torch.full_like(x, 1) for x in whole]
        torch.cuda.synchronize()
        _same(_np(one), ref_one, "one group")
        _same(_np(many[0]), _np(ref_all[0]), "start messages")
        del junk


def test_buffers_of_a_side_stream_call_are_its_own(dev):
    """Calls on a side stream that allocate their workspace and outputs, the current stream's allocator having just
    got blocks of those sizes back: with the current stream behind (its last writes to those blocks are still to come)
    and with the side stream behind (the call has dropped its workspace before running), results equal those of the
    idle device and memory allocated afterwards keeps what is written to it."""
    import torch
    import paper_2402_04834_amd as bbp
    from paper_2402_04834_amd import warm
    d, b = 9, 24
    opts = bbp.default_opts(block=6, chi=32, max_iter=8)
    syn = torch.from_numpy(workload.make_batch(d, 0.1, b, workload="test", p_index=79)[1]).to(dev)
    prm = torch.from_numpy(warm.init_params(5)).to(dev)
    st = torch.cuda.Stream(dev)
    predict = lambda **kw: dict(messages=warm.predict(d, 0.1, syn, opts, prm, **kw))
    decode = lambda **kw: {k: v for k, v in bbp.decode_device(d, 0.1, syn, opts, **kw).items() if k in KEYS}
    for name, call, ws_bytes in (("predict", predict, warm.workspace_size(d, b, opts, False)),
                                 ("decode", decode, bbp.workspace_size(d, b, opts))):
        ref = {k: v.clone() for k, v in call().items()}
        torch.cuda.synchronize()
        sizes = [ws_bytes] + [v.numel() * v.element_size() for v in ref.values()]
        for behind in ("current", "side"):
            _say(f"[side stream buffers] {name}, the {behind} stream behind")
            blocks = [torch.empty(n, dtype=torch.uint8, device=dev) for n in sizes]
            torch.cuda.synchronize()
            if behind == "current":
                torch.cuda._sleep(20_000_000)
                for n in range(len(blocks)):
                    blocks[n].fill_(255)
            else:
                with torch.cuda.stream(st):
                    torch.cuda._sleep(20_000_000)
            del blocks
            got = call(stream=st)
            after = [torch.full((n,), 85, dtype=torch.uint8, device=dev) for n in sizes]
            torch.cuda.synchronize()
            for key, v in ref.items():
                assert torch.equal(got[key].view(torch.uint8), v.view(torch.uint8)), key
            assert all(bool((x == 85).all()) for x in after)
            del after


@pytest.mark.parametrize("d,k", [(5, 2), (7, 1)])
def test_autotune_times_class_launches(dev, d, k):
    """The launch variants are variants of the class launches: tuning on a batch that decodes in one launch (5 to 20
    times as fast here) times the class launches all the same, whose launches alone, timed one by one, take at most four
    times as long as the decode that overlaps them."""
    import torch
    import paper_2402_04834_amd as bbp
    _, syn = workload.make_batch(d, 0.1, 2, workload="test", p_index=180 + d)
    s = torch.from_numpy(syn).to(dev)
    opts = bbp.default_opts(block=k, chi=32, fixed_iters=1)
    try:
        for _ in range(2):
            tm = bbp.decode_device(d, 0.1, s, opts, timing=True)["timing"]
        best = bbp.autotune(d, 0.1, s, opts)
        _say(f"[autotune] d={d} k={k}: launches {tm.update_ms + tm.bethe_ms + tm.other_ms:.3f} ms, tuned {best.ms:.3f} ms")
        assert best.ms > 0.25 * (tm.update_ms + tm.bethe_ms + tm.other_ms)
    finally:
        bbp.set_tuning(d, opts, 0, 1)


# batches beyond the smaller routes' reach; packed widths (blocks 3 to 5) with a last job block that is partly filled
CLASS_BATCHES = [(5, 3, 2501, 0), (5, 4, 3501, 1), (6, 5, 2501, 0), (9, 6, 1501, 1)]


@pytest.mark.parametrize("d,k,b,precision", CLASS_BATCHES)
def test_launch_variants_of_class_launches(dev, d, k, b, precision):
    """Decodes by class launches, item order sweep-major and job-major, on 1, 2 and 4 streams, eager and as a graph
    replayed with other work between, equal the first variant's bitwise, and its first syndromes decoded by themselves."""
    import torch
    import paper_2402_04834_amd as bbp
    p = 0.10
    opts = bbp.default_opts(block=k, chi=32, max_iter=6, precision=precision)
    graph = bbp.default_opts(block=k, chi=32, max_iter=6, precision=precision, graph=1)
    assert bbp.launch_route([(d, b)], opts) == 0 and bbp.launch_route([(d, b)], graph) == 0
    _, syn = workload.make_batch(d, p, b, workload="mixed", p_index=130 + d)
    s = torch.from_numpy(syn).to(dev)
    st = torch.cuda.Stream(dev)
    ws = torch.empty(bbp.workspace_size(d, b, opts), dtype=torch.uint8, device=dev)
    ref, out = None, None
    try:
        for order in (0, 1):
            for streams in (1, 2, 4):
                _say(f"[class variants] d={d} k={k} batch {b} order={order} streams={streams}")
                bbp.set_tuning(d, opts, order, streams)
                got = _alone(dev, d, p, syn, opts)
                ref = got if ref is None else ref
                _same(got, ref, f"order {order} streams {streams}")
                for replay in range(3 if streams > 1 else 0):
                    out = bbp.decode_device(d, p, s, graph, workspace=ws, stream=st, out=out)
                    st.synchronize()
                    _same(_np(out), ref, f"graph {replay}, order {order} streams {streams}")
                    for key in KEYS:
                        out[key].zero_()
                    torch.cuda.synchronize()
    finally:
        bbp.set_tuning(d, opts, 0, 1)
    few = _alone(dev, d, p, syn[:3], opts)
    _same(few, {key: ref[key][:3] for key in KEYS}, "first syndromes")


def test_concurrent_multistream_class_launches(dev):
    """Two host threads whose decodes spread class launches over the device's auxiliary streams, eagerly and through
    captured graphs, each on its own stream: every result is bitwise the single-stream decode's."""
    import threading
    import torch
    import paper_2402_04834_amd as bbp
    d, p, b = 9, 0.10, 1501
    opts, gopts = (bbp.default_opts(block=6, chi=32, max_iter=6, graph=g) for g in (0, 1))
    assert bbp.launch_route([(d, b)], opts) == 0 and bbp.launch_route([(d, b)], gopts) == 0
    syn = [torch.from_numpy(workload.make_batch(d, p, b, workload="mixed", p_index=140 + k)[1]).to(dev) for k in range(2)]
    bbp.set_tuning(d, opts, 0, 1)
    ref = [_np(bbp.decode_device(d, p, s, opts)) for s in syn]
    bbp.set_tuning(d, opts, 1, 4)
    errors, done = [], [0, 0]

    def worker(k):
        try:
            st = torch.cuda.Stream(dev)
            ws = torch.empty(bbp.workspace_size(d, b, opts), dtype=torch.uint8, device=dev)
            out = None
            for rep in range(6):
                out = bbp.decode_device(d, p, syn[k], gopts if rep % 2 else opts, workspace=ws, stream=st, out=out)
                st.synchronize()
                _same(_np(out), ref[k], f"thread {k} decode {rep}")
                done[k] += 1
        except BaseException as e:   # reported by the main thread
            errors.append(e)

    _say("[concurrent class launches] two threads, 4-stream variant, eager and graph")
    try:
        th = [threading.Thread(target=worker, args=(k,)) for k in range(2)]
        for t in th:
            t.start()
        for t in th:
            t.join()
        assert not errors, errors
        assert done == [6, 6]
    finally:
        bbp.set_tuning(d, opts, 0, 1)
