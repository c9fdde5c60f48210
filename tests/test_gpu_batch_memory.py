"""What a batch's handle keeps is bounded by the caller (KNN_SPLIT_BYTES), with the
same results."""
import os

import pytest
import torch

pytestmark = pytest.mark.gpu


def test_operands_within_the_callers_limit():
    import paper_1309_5478_amd as knn
    g = torch.Generator(device="cuda")
    g.manual_seed(4)
    C = torch.randn((200000, 512), generator=g, device="cuda")     # 0.38 GiB of operands a job
    Q = torch.randn((160, 512), generator=g, device="cuda")
    jobs = [(Q, C, 5)] * 8

    def kept(limit):
        if limit is not None:
            os.environ["KNN_SPLIT_BYTES"] = str(limit)
        try:
            h = knn.Handle(0)
            torch.cuda.synchronize()
            out = [(torch.empty((160, 5), device="cuda"), torch.empty((160, 5), dtype=torch.int32, device="cuda"))
                   for _ in jobs]
            before = torch.cuda.mem_get_info()[0]
            h.batch_search(jobs, out=out)
            torch.cuda.synchronize()
            return before - torch.cuda.mem_get_info()[0], out
        finally:
            os.environ.pop("KNN_SPLIT_BYTES", None)
    free, a = kept(None)
    half, b = kept(4 * (200000 + 160 + 16384) * 512 * 4)          # four of eight, each with its queries and sample
    none, c = kept(1)
    one = 200000 * 512 * 4
    print(f"kept: {free >> 20}, {half >> 20}, {none >> 20} MiB", flush=True)
    assert free - half >= 3.9 * one and half - none >= 3.9 * one
    for x, y, z in zip(a, b, c):
        for s, t, u in zip(x, y, z):
            assert torch.equal(s, t) and torch.equal(s, u)
