"""The clustering call under a HIP graph.  The row sort hands its units of work out from a counter that the last
workgroup of a launch leaves at zero; a captured launch must find it so on every replay, also with eager calls of
the same context in between.  Replays are checked against the eager result, bit for bit (same kernels, same inputs:
the results do not depend on which workgroup sorted a row)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_error_table_replays_from_a_captured_graph(gpu_lib):
    stream = torch.cuda.Stream()
    ctx = gpu_lib.Context(0, stream=stream)
    try:
        # more rows than workgroups resident at once (two per compute unit at this length): most units are claimed
        n, m = 1500, 4096
        rng = np.random.default_rng(812)
        W = (rng.standard_normal((n, m)) * 0.02).astype(np.float32)
        S = (rng.standard_normal((n, m)) ** 2).astype(np.float32)
        W2 = (rng.standard_normal((n, m)) * 0.05).astype(np.float32)
        with torch.cuda.stream(stream):
            Wd, Sd, W2d = torch.from_numpy(W).cuda(), torch.from_numpy(S).cuda(), torch.from_numpy(W2).cuda()
            eager = ctx.error_table(Wd, Sd)
            out = {k: torch.empty_like(v) for k, v in eager.items()}
            other = ctx.error_table(W2d, Sd)
        stream.synchronize()
        ref = {k: v.clone() for k, v in eager.items()}
        ref_other = {k: v.clone() for k, v in other.items()}
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            ctx.error_table(Wd, Sd, out=out)
        for rep in range(4):
            with torch.cuda.stream(stream):
                for v in out.values():
                    v.zero_()
                ctx.error_table(W2d, Sd, out=other)      # eager work of the same context between the replays
                graph.replay()
            stream.synchronize()
            for k in ref:
                assert torch.equal(out[k], ref[k]), f"replay {rep}: {k} differs from the eager call"
                assert torch.equal(other[k], ref_other[k]), f"replay {rep}: eager {k} changed"
    finally:
        ctx.close()


def test_hessian_leaves_the_memory_of_captured_calls_alone(gpu_lib):
    """A captured call holds the addresses of the context's buffers.  A Hessian that needs more scratch than any before it
    must not have the allocator hand those to others: neither the workspace of a captured clustering, nor the scratch of a
    captured Hessian (also not when the workspace grows)."""
    stream = torch.cuda.Stream()
    ctx = gpu_lib.Context(0, stream=stream)
    try:
        gen = torch.Generator(device="cuda").manual_seed(3)
        with torch.cuda.stream(stream):
            W = torch.randn((64, 512), device="cuda", generator=gen)
            S = torch.rand((64, 512), device="cuda", generator=gen)
            X = torch.randn((1024, 130), device="cuda", generator=gen).to(torch.bfloat16)
            Xbig = torch.randn((8192, 1536), device="cuda", generator=gen).to(torch.bfloat16)
            eager = ctx.error_table(W, S)
            H = ctx.hessian_from_activations(X)
            ref = {k: v.clone() for k, v in eager.items()}
            ref_H = H.clone()
        stream.synchronize()
        ws, blocks = ctx._ws, list(ctx._hessian_blocks)
        assert len(blocks) == 1
        table_graph, hessian_graph = torch.cuda.CUDAGraph(), torch.cuda.CUDAGraph()
        with torch.cuda.graph(table_graph, stream=stream):
            ctx.error_table(W, S, out=eager)
        with torch.cuda.graph(hessian_graph, stream=stream):
            ctx.hessian_from_activations(X, out=H)
            ctx.hessian_from_activations(Xbig)          # (more than there is: runs without scratch, allocates none)
        assert ctx._ws is ws and ctx._hessian_blocks == blocks
        big = ctx.hessian_from_activations(Xbig)        # a larger block
        assert ctx._ws is ws, "the Hessian replaced the registered workspace"
        assert len(ctx._hessian_blocks) == 2 and ctx._hessian_blocks[0] is blocks[0]
        for rep in range(3):
            with torch.cuda.stream(stream):
                # whatever the allocator would hand out of blocks that went back to it
                others = [torch.full((n,), 7, dtype=torch.uint8, device="cuda") for n in (ws.numel(), blocks[0].numel())]
                for v in list(eager.values()) + [H]:
                    v.zero_()
                table_graph.replay()
                hessian_graph.replay()
                again = ctx.hessian_from_activations(Xbig)
            stream.synchronize()
            for k in ref:
                assert torch.equal(eager[k], ref[k]), f"replay {rep}: {k}"
            assert torch.equal(H, ref_H) and torch.equal(again, big), f"replay {rep}"
            assert all(bool((t == 7).all()) for t in others), f"replay {rep}: another tensor was written"
    finally:
        ctx.close()
