"""The uploads' kernel copies tables whole, on both sides of the end of its workgroups: a launch over many tensors or jobs
against one launch for each."""
import numpy as np
import pytest
import torch

from test_gpu_schedules import launch, model

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2604_06836_amd as stq
    c = stq.Context(0, 64)
    yield c
    c.close()


# a workgroup copies 4096 bytes: 42 tensors of 96 bytes and two thirds of another
@pytest.mark.parametrize("n", [1, 42, 43, 64])
def test_tensor_tables(ctx, n):
    sizes = [1 + (977 * l) % 5000 for l in range(n)]
    plan = [(2 + l % 7, 2 + l % 5) for l in range(n)]
    got = []
    for together in (False, True):
        m = model(ctx, sizes, plan, 64, 91, "fp32")
        m.set_grads(1)
        for t in (1, 2):
            for g in [list(range(n))] if together else [[l] for l in range(n)]:
                launch(ctx, m, t, g, None, False)
        torch.cuda.synchronize()
        codes = [[buf[l][:m._code_words(sizes[l], plan[l][k])] for l in range(n)] for k, buf in enumerate((m.m_codes, m.v_codes))]
        got.append([m.param, m.m_scales, m.v_scales, *codes])
    for a, b in zip(*got):
        for l, (x, y) in enumerate(zip(a, b)):
            assert torch.equal(x.view(torch.int32), y.view(torch.int32)), l


# 48 bytes a job: 85 and a third
@pytest.mark.parametrize("n", [1, 85, 86, 128])
def test_job_tables(ctx, n):
    s = torch.cuda.current_stream().cuda_stream
    rng = np.random.default_rng(92)
    src, dst, jobs = [], [[], []], []
    for l in range(n):
        numel, b0, b1 = 1 + (977 * l) % 5000, int(rng.integers(2, 9)), int(rng.integers(2, 9))
        tiles = (numel + 2047) // 2048
        src.append(torch.from_numpy(rng.integers(-2 ** 31, 2 ** 31, tiles * 64 * b0).astype(np.int32)).to("cuda:0"))
        for d in dst:
            d.append(torch.full((tiles * 64 * b1,), -1, device="cuda:0", dtype=torch.int32))
        jobs.append((numel, l % 2, src[l].data_ptr(), b0, b1))
    ctx.repack_many([(k, st, p, b0, d.data_ptr(), b1) for (k, st, p, b0, b1), d in zip(jobs, dst[0])], 64, s)
    for (k, st, p, b0, b1), d in zip(jobs, dst[1]):
        ctx.repack(k, 64, st, p, b0, d.data_ptr(), b1, s)
    torch.cuda.synchronize()
    for l, (x, y) in enumerate(zip(*dst)):
        assert torch.equal(x, y), l


@pytest.mark.parametrize("kind", ["step", "repack", "engine", "engine-481"])
def test_sixteen_uploads_ahead_of_the_device(kind):
    """Sixteen calls that upload a table each return while the stream is still busy with earlier work, whichever staging slot
    they begin at, and their results are those of calls that were waited for.  (An engine of up to 480 tensors has no slots: its
    addresses are the launch's arguments.)"""
    import paper_2604_06836_amd as stq
    from paper_2604_06836_amd import binding
    from workloads.harness import hparams
    sizes = [700, 2049, 5] if kind != "engine-481" else [1 + (977 * l) % 300 for l in range(481)]
    n, K, got = len(sizes), 64, []
    for ahead in (False, True):
        c = stq.Context(0, 512 if n > 8 else 8)
        m = model(c, sizes, [(4, 4)] * n, K, 93, "fp32")
        for lst in (m.m_codes, m.v_codes):  # nothing undefined behind the codes
            for l, buf in enumerate(lst):
                buf[m._code_words(m.numel[l], 4):] = 0
        grads = []
        for k in range(7):
            m.set_grads(k + 1)
            grads.append([g.clone() for g in m.grad])
        addresses = [[g.data_ptr() for g in gs] for gs in grads]
        out = [[torch.zeros_like(m.m_codes[l]) for l in range(n)] for _ in range(17 if kind == "repack" else 0)]
        eng = None
        if kind.startswith("engine"):
            eng = c.engine(m.tensors, [(m._spare[(l, 0)].data_ptr(), m._spare[(l, 1)].data_ptr()) for l in range(n)], m.cplan, 8, K,
                           thr=(6.8,), bits=(4, 8), stream=m.stream)

        def call(k, t):
            if kind.startswith("engine"):  # (no decisions: past the first steps)
                eng.step(hparams(m.w, t), 0, addresses[t % 7], m.stream)
            elif kind == "repack":
                c.repack_many([(m.numel[l], 0, m.m_codes[l].data_ptr(), 4, out[k][l].data_ptr(), 2 + t % 7) for l in range(n)], K, m.stream)
            else:  # 21 argument sets in turn, more than there are tables
                which = ([0, 1, 2], [0, 1], [1, 2])[t % 3]
                sub = (binding.Tensor * len(which))(*[m.tensors[l] for l in which])
                for x, l in zip(sub, which):
                    x.grad = grads[t % 7][l].data_ptr()
                c.step(sub, binding.make_plan([m.plan[l] for l in which]), hparams(m.w, t), m.stream)

        for phase in range(24):  # 17 uploads each, so that every slot is the first of the sixteen once
            if ahead:
                torch.cuda._sleep(10_000_000)  # some milliseconds or more
                busy = torch.cuda.Event()
                busy.record()
            for k in range(17):
                if ahead and k == 16:
                    assert not busy.query(), phase
                if not ahead or k == 16:
                    torch.cuda.synchronize()
                call(k, 5 + 17 * phase + k)
            torch.cuda.synchronize()
        got.append([x.view(torch.int32).clone() for x in [*m.param, *m.m_codes, *m.v_codes, *m.m_scales, *m.v_scales, *sum(out, [])]])
        if eng:
            eng.close()
        c.close()
    for l, (x, y) in enumerate(zip(*got)):
        assert torch.equal(x, y), l


# Up to 480 addresses of gradients travel in the launch's arguments, more through a staging slot.  (Eleven uploads: the slots come
# round in test_sixteen_uploads_ahead_of_the_device.)
@pytest.mark.parametrize("n", [1, 480, 481])
def test_addresses_of_the_gradients(n):
    import paper_2604_06836_amd as stq
    from workloads.harness import hparams
    sizes, K, got = [1 + (977 * l) % 300 for l in range(n)], 64, []
    for by_address in (False, True):
        c = stq.Context(0, 512)
        m = model(c, sizes, [(4, 4)] * n, K, 94, "fp32")
        for lst in (m.m_codes, m.v_codes):
            for l, buf in enumerate(lst):
                buf[m._code_words(sizes[l], 4):] = 0
        for x in m._spare.values():
            x.zero_()
        eng = c.engine(m.tensors, [(m._spare[(l, 0)].data_ptr(), m._spare[(l, 1)].data_ptr()) for l in range(n)], m.cplan, 8, K,
                       thr=(6.8,), bits=(4, 8), stream=m.stream)
        grads = []
        for k in range(3):
            m.set_grads(k + 1)
            grads.append([g.clone() for g in m.grad])
        for t in range(1, 31):  # (decisions up to step 4; two of three steps keep the addresses they have)
            g = grads[(t - t % 3) % 9 // 3]
            if by_address:
                eng.step(hparams(m.w, t), 0, [x.data_ptr() for x in g] if t % 3 == 0 or t == 1 else None, m.stream)
            else:
                for x, y in zip(m.grad, g):
                    x.copy_(y)
                eng.step(hparams(m.w, t), 0, None, m.stream)
        torch.cuda.synchronize()
        spare = [m._spare[k] for k in sorted(m._spare)]
        got.append([x.view(torch.int32).clone() for x in [*m.param, *m.m_codes, *m.v_codes, *spare, *m.m_scales, *m.v_scales]])
        eng.close()
        c.close()
    for l, (x, y) in enumerate(zip(*got)):
        assert torch.equal(x, y), l
