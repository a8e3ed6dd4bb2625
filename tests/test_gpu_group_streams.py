"""Transform groups on several streams: that they fork where the size rule says
so (seen in the captured graph of an operator), and that a batch whose groups
are compacted inside captured chunks gives one stream's bits."""
import re

import pytest

from paper_1710_00621_amd import inputs

pytestmark = pytest.mark.gpu


def _model(crsolve, scale):
    prob = inputs.make_problem("multires", scale=scale)
    taus = inputs.inverse_noise_maps(prob, lambda spec: crsolve.Grid.from_spec(spec).pixel_centres())
    return crsolve.model_from_problem(prob, taus)


def _branches(dot):
    """The largest number of edges that leave one node of a graph in dot form."""
    out = {}
    for a, b in re.findall(r'"([^"]+)"\s*->\s*"([^"]+)"', dot):
        out.setdefault(a, set()).add(b)
    assert out, dot[:400]
    return max(len(v) for v in out.values())


@pytest.mark.parametrize("scale,env,branches", [(2, None, 3), (2, "1", 1), (2, "2", 2), (8, None, 1)])
def test_groups_fork_where_they_are_large(scale, env, branches, monkeypatch, tmp_path):
    import torch
    from paper_1710_00621_amd import crsolve
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    print(f"case group streams scale {scale} CRS_GROUP_STREAMS={env}", flush=True)
    monkeypatch.delenv("CRS_GROUP_STREAMS", raising=False)
    if env:
        monkeypatch.setenv("CRS_GROUP_STREAMS", env)
    gm = _model(crsolve, scale)
    gen = torch.Generator(device="cpu").manual_seed(97)
    x = torch.randn(1, gm.n, generator=gen, dtype=torch.float64).to("cuda")
    ref = gm.apply_A(x)  # builds the operator's state and its streams
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph(keep_graph=True)
    g.enable_debug_mode()
    with torch.cuda.graph(g):
        y = gm.apply_A(x)
    path = tmp_path / "graph.dot"
    g.debug_dump(str(path))
    assert _branches(path.read_text()) == branches
    for _ in range(3):
        y.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, ref)
        assert torch.equal(gm.apply_A(x), ref)


def test_batch_of_many_maps_per_group_bitwise(monkeypatch):
    """Ten problems share their grids, so that every group has more than eight
    maps and its launches take lists of the active ones."""
    import torch
    from paper_1710_00621_amd import crsolve
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    print("case batch of ten on the rule's streams and on one", flush=True)
    monkeypatch.delenv("CRS_GROUP_STREAMS", raising=False)
    prob = inputs.make_problem("multires", scale=2)
    grids = {b["grid"]: crsolve.Grid.from_spec(b["grid"]) for b in prob["bands"]}
    gl = [grids[b["grid"]] for b in prob["bands"]]
    taus = inputs.inverse_noise_maps(prob, lambda spec: grids[spec].pixel_centres())
    models = [crsolve.model_from_problem(prob, taus, gl) for _ in range(10)]
    gen = torch.Generator(device="cpu").manual_seed(101)
    data = [[torch.randn(g.npix, generator=gen, dtype=torch.float64).to("cuda") * (1.0 + 9.0 * (p > 4))
             for g in gl] for p in range(10)]
    out = []
    batch = crsolve.Batch(models)  # one batch: it tunes its own tiles
    for streams in (None, 1):
        if streams:
            batch.set_streams(streams)
        x, info = batch.solve(d=data, seeds=list(range(10)), mode="cr", precond="pinv", rtol=1e-8, maxiter=40,
                              use_graph=True, raise_on_error=False)
        out.append(([t.cpu() for t in x], list(info["iters"])))
    (xa, ia), (xb, ib) = out
    assert ia == ib
    for a, b in zip(xa, xb):
        assert torch.equal(a, b)
