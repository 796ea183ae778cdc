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
