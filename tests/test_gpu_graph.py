"""A step whose tensor table is already on the device is kernel launches only, so a caller can record it into
a HIP graph: recorded here through torch's stream capture, replayed several times with eager work and
synchronisations of the program in between, and every replay compared with the eager run of the same calls
(a recorded launch repeats the step number it was recorded with).  Both schedules: the ticket counter has to
reset itself between replays, since nothing outside the kernel touches it."""
import numpy as np
import pytest
import torch

import paper_2604_06836_amd as stq
from workloads import configs
from workloads.harness import DeviceModel, hparams

pytestmark = pytest.mark.gpu


def snapshot(dm):
    return [tuple(a.copy() for a in dm.host_state(l)) for l in range(len(dm.numel))]


def same(a, b, tag):
    for l, (x, y) in enumerate(zip(a, b)):
        for name, u, v in zip(("param", "m codes", "m scales", "v codes", "v scales"), x, y):
            assert np.array_equal(u.view(np.uint32), v.view(np.uint32)), f"{tag}: tensor {l} {name}"


@pytest.mark.parametrize("tickets,kind", [(False, "grad"), (True, "grad"), (True, True)])
def test_recorded_step_replays_like_the_eager_step(tickets, kind):
    w = configs.Workload(85, "graph", [("a", 30 * 2048 + 99), ("b", 4097), ("c", 12 * 2048)], 128, "bf16", 1,
                         "normal_per_tensor")
    plan = [(5, 4), (8, 3), (4, 6)]
    side = torch.cuda.Stream()
    ctxs = [stq.Context(0, 8), stq.Context(0, 8)]
    try:
        for c in ctxs:
            c.set_schedule(1 if tickets else 2 ** 63)
        with torch.cuda.stream(side):   # DeviceModel takes the current stream: everything on `side`
            ref, rec = DeviceModel(ctxs[0], w, plan), DeviceModel(ctxs[1], w, plan)
            for dm in (ref, rec):
                dm.set_grads(1)
                dm.step(1)              # uploads the tensor table on this stream
            side.synchronize()
            same(snapshot(ref), snapshot(rec), "before recording")
            hp = hparams(w, 2, kind)    # the recorded step also gathers statistics: the gradient's, or all
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=side):
                rec.ctx.step(rec.tensors, rec.cplan, hp, side.cuda_stream)
            for replay in range(4):
                graph.replay()
                ref.ctx.step(ref.tensors, ref.cplan, hp, side.cuda_stream)
                side.synchronize()
                same(snapshot(ref), snapshot(rec), f"replay {replay}")
                # eager work of the program between the replays
                junk = torch.ones(1 << 20, device="cuda")
                junk.mul_(2.0)
                side.synchronize()
            a, b = ref.ctx.stats(3, side.cuda_stream), rec.ctx.stats(3, side.cuda_stream)
            # (the recorded launches are not counted by the host: their statistics are read as one step's)
            for l in range(3):
                assert abs(a[l].g_sq_sum - b[l].g_sq_sum) <= 1e-12 * a[l].g_sq_sum and a[l].g_absmax == b[l].g_absmax
                assert abs(a[l].m_sq_sum - b[l].m_sq_sum) <= 1e-6 * a[l].m_sq_sum and a[l].v_absmax == b[l].v_absmax
                assert (a[l].m_sq_sum > 0) == (kind is True)
    finally:
        for c in ctxs:
            c.close()


# Calls that bring a table with them: recorded, then many calls of the same kind with tables of their own (as many as there are
# staging slots and more), then replays.  Everything else in the two contexts is alike, call for call.  The other calls' tables
# have the same sizes.  90 tensors: two launches' arguments and a part of a third; 500: two of gradient addresses.
def uploading_models(ctx, n, seed):
    w = configs.Workload(seed, "graph", [("t%d" % l, 1 + (977 * l) % 3000) for l in range(n)], 64, "fp32", 1, "normal_per_tensor")
    dm = DeviceModel(ctx, w, [(2 + l % 7, 2 + l % 5) for l in range(n)], spare_width=8)
    for lst in (dm.m_codes, dm.v_codes):
        for l, buf in enumerate(lst):
            buf[dm._code_words(dm.numel[l], dm.plan[l][0 if lst is dm.m_codes else 1]):] = 0
    for s in dm._spare.values():
        s.zero_()
    dm.set_grads(1)
    return dm


def buffers(dm):
    lists = (dm.param, dm.m_scales, dm.v_scales, dm.m_codes, dm.v_codes)
    return [t.view(torch.int32).clone() for lst in lists for t in lst] + [t.clone() for t in dm._spare.values()]


class Uploading:
    """One kind of call on a context, with a model of its own for every set of arguments."""

    def __init__(self, kind, n, stream):
        self.kind, self.n, self.s = kind, n, stream.cuda_stream
        self.ctx = stq.Context(0, 512)
        self.dm, self.other = uploading_models(self.ctx, n, 86), [uploading_models(self.ctx, n, 87 + k) for k in range(2 if kind == "engine" else 6)]
        if kind == "engine":
            dm = self.dm
            second = [(dm._spare[(l, 0)].data_ptr(), dm._spare[(l, 1)].data_ptr()) for l in range(n)]
            self.eng = self.ctx.engine(dm.tensors, second, dm.cplan, 8, 64, thr=(6.8,), bits=(4, 8), stream=self.s)

    def call(self, dm, t):
        if self.kind == "step":
            self.ctx.step(dm.tensors, dm.cplan, hparams(dm.w, t), self.s)
        elif self.kind == "static":
            self.ctx.step_static(dm.tensors, dm.cplan, hparams(dm.w, t), self.s)
        elif self.kind == "grad":
            self.ctx.grad_stats(dm.tensors, 64, 0, self.s)
        elif self.kind == "engine":  # (a step without a decision)
            self.eng.step(hparams(self.dm.w, t + 4), 0, [g.data_ptr() for g in dm.grad], self.s)
        else:
            new = [(2 + (m + l) % 7, 2 + (v + l) % 7) for l, (m, v) in enumerate(dm.plan)]
            if self.kind == "transition":
                dst = [tuple(dm._spare[(l, k)].data_ptr() if new[l][k] != dm.plan[l][k] else None for k in (0, 1)) for l in range(self.n)]
                self.ctx.step_transition(dm.tensors, dm.cplan, stq.binding.make_plan(new), dst, hparams(dm.w, t), self.s)
            else:
                self.ctx.repack_many([(dm.numel[l], k, cur[l].data_ptr(), dm.plan[l][k], dm._spare[(l, k)].data_ptr(), new[l][k])
                                      for l in range(self.n) for k, cur in ((0, dm.m_codes), (1, dm.v_codes))], 64, self.s)

    def results(self):
        torch.cuda.synchronize()
        out = [b for dm in [self.dm] + self.other for b in buffers(dm)]
        if self.kind == "grad":
            out.append(torch.tensor([(s.g_sum, s.g_abs_sum, s.g_sq_sum, s.g_absmax) for s in self.ctx.stats(self.n, self.s)], dtype=torch.float64))
        return out


def same_results(a, b, tag):
    for l, (x, y) in enumerate(zip(a, b)):
        if x.dtype != torch.float64:
            assert torch.equal(x, y), (tag, l)
        else:  # sums in fp64 in another order: n * 2^-53 of the sum of absolute values, n <= 3000
            assert torch.equal(x[:, 3], y[:, 3]) and (x[:, 3] > 0).all(), tag
            assert ((x - y)[:, :2].abs() <= 1e-12 * x[:, 1:2]).all() and ((x - y)[:, 2].abs() <= 1e-12 * x[:, 2]).all(), tag


@pytest.mark.parametrize("kind,n", [("step", 3), ("step", 90), ("transition", 90), ("static", 3), ("static", 90), ("grad", 90), ("repack", 90),
                                    ("engine", 3), ("engine", 500)])
def test_recorded_uploads_outlive_the_calls_that_follow(kind, n):
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        ref, rec = Uploading(kind, n, side), Uploading(kind, n, side)
        try:
            side.synchronize()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=side):
                rec.call(rec.dm, 7)
            if kind != "grad":
                same_results(ref.results(), rec.results(), "recording alone does nothing")
            for replay in range(3):
                for u in (ref, rec):  # 40 uploads
                    for k in range(40):
                        u.call(u.other[k % len(u.other)], 8 + k)
                if kind == "grad":  # clear the accumulators: what follows is the recorded call's, and a count for it
                    for u in (ref, rec):
                        u.ctx.stats(n, u.s)
                        for g in u.other[0].grad:
                            g.zero_()
                        u.call(u.other[0], 1)
                graph.replay()
                ref.call(ref.dm, 7)
                same_results(ref.results(), rec.results(), replay)
                junk = torch.ones(1 << 20, device="cuda")  # eager work of the program between the replays
                junk.mul_(2.0)
                side.synchronize()
        finally:
            for u in (ref, rec):
                if kind == "engine":
                    u.eng.close()
                u.ctx.close()


def test_a_table_that_was_only_recorded_is_uploaded_by_the_next_call():
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        ref, rec = Uploading("step", 3, side), Uploading("step", 3, side)
        try:
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=side):
                rec.call(rec.dm, 1)
            for u in (ref, rec):
                u.call(u.dm, 1)
            same_results(ref.results(), rec.results(), "the eager call")
        finally:
            for u in (ref, rec):
                u.ctx.close()


def test_recorded_launches_keep_their_resident_tables():
    """Six argument sets that are on the device when they are recorded (more than the context holds for recordings), then calls
    with more other sets than there are tables, then replays."""
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        ref, rec = Uploading("step", 3, side), Uploading("step", 3, side)
        others = [uploading_models(ref.ctx, 3, 95 + k) for k in range(9)], [uploading_models(rec.ctx, 3, 95 + k) for k in range(9)]
        try:
            graphs = [torch.cuda.CUDAGraph() for _ in range(6)]
            for k, graph in enumerate(graphs):
                for u in (ref, rec):
                    u.call(u.other[k], 1)  # eager: uploads the table
                with torch.cuda.graph(graph, stream=side):
                    rec.call(rec.other[k], 2)
            for replay in range(2):
                for u, more in zip((ref, rec), others):
                    for _ in range(2):
                        for dm in more:
                            u.call(dm, 3)
                for k, graph in enumerate(graphs):
                    graph.replay()
                    ref.call(ref.other[k], 2)
                same_results(ref.results(), rec.results(), replay)
                for a, b in zip(*others):
                    same_results(buffers(a), buffers(b), replay)
        finally:
            for u in (ref, rec):
                u.ctx.close()


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("alg1", [False, True])
def test_recorded_steps_of_the_loop(alg1, wide):
    """Steps with and without a decision, recorded while one was waiting or not, replayed in an order of their own among eager
    steps: the same as the eager calls."""
    bits = (4, 8, 16, 32) if wide else (3, 4, 6, 8)
    side = torch.cuda.Stream()
    sizes = [700, 2048 * 3, 5000, 9, 4097, 2048 * 2 + 1]
    with torch.cuda.stream(side):
        s = side.cuda_stream
        both = []
        for _ in range(2):
            ctx = stq.Context(0, 8)
            w = configs.Workload(97, "loop", [("t%d" % l, n) for l, n in enumerate(sizes)], 64, "fp32", 1, "normal_per_tensor")
            dm = DeviceModel(ctx, w, [(4, 8)] * len(sizes), spare_width=32)
            grads = []
            for k in range(2):
                dm.set_grads(k + 1)
                grads.append([g.clone() for g in dm.grad])
            second = [(dm._spare[(l, 0)].data_ptr(), dm._spare[(l, 1)].data_ptr()) for l in range(len(sizes))]
            eng = ctx.engine(dm.tensors, second, dm.cplan, 32, 64, thr=(8.0, 11.0, 14.0), bits=bits, alg1_order=alg1, stream=s)
            both.append((ctx, dm, eng, grads))
        by_ptr = [{b.data_ptr(): b for b in [*dm.m_codes, *dm.v_codes, *dm._spare.values()]} for _, dm, _, _ in both]
        widths = set()

        def step(i, t, every, k):
            _, dm, eng, grads = both[i]
            eng.step(hparams(dm.w, t), every, [g.data_ptr() for g in grads[k]], s)

        def check(tag):
            side.synchronize()
            a, b = (eng.read(s) for _, _, eng, _ in both)
            assert a["stored"] == b["stored"] and a["next"] == b["next"], tag
            widths.update(a["stored"])
            for l, n in enumerate(sizes):
                for k in (0, 1):
                    words = both[0][1]._code_words(n, a["stored"][l][k])
                    assert torch.equal(by_ptr[0][a["current"][l][k]][:words], by_ptr[1][b["current"][l][k]][:words]), (tag, l, k)
                for x, y in ((both[i][1] for i in (0, 1)),):
                    for name in ("param", "m_scales", "v_scales"):
                        assert torch.equal(getattr(x, name)[l].view(torch.int32), getattr(y, name)[l].view(torch.int32)), (tag, l, name)

        try:
            graphs = {}

            def record(name, t, every, k):
                graphs[name] = (torch.cuda.CUDAGraph(), t, every, k)
                with torch.cuda.graph(graphs[name][0], stream=side):
                    step(1, t, every, k)

            def replay(name):
                graph, t, every, k = graphs[name]
                graph.replay()
                step(0, t, every, k)

            def eager(*a):
                step(0, *a)
                step(1, *a)

            record("plain", 11, 0, 0)             # nothing waits
            eager(10, 10, 0)                      # a decision, which then waits (default order)
            record("waiting", 12, 0, 1)
            eager(13, 0, 0)                       # takes it, though the recorded step came first
            check("eager")
            eager(20, 10, 1)
            if alg1 or wide:                      # (a recorded in-place step leaves the decision waiting, which no eager step does)
                replay("plain")
            replay("waiting")
            check("a waiting decision")
            record("decides", 30, 10, 1)
            for n in range(3):
                replay("decides")
                check("decides %d" % n)
            eager(31, 0, 0)
            check("eager after a replayed decision")
            replay("decides")
            eager(40, 10, 0)
            replay("waiting")
            check("a decision after a replayed one")
            replay("decides")
            replay("decides")
            eager(41, 0, 1)
            eager(42, 0, 1)
            replay("plain")
            check("end")
            assert len(widths) > 2, widths
        finally:
            for ctx, _, eng, _ in both:
                eng.close()
                ctx.close()
