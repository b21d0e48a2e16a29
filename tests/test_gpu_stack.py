"""Stack calls that run phase by phase (four or more consecutive layers of one shape): selections,
products and reductions of all layers in one launch each, against per-layer calls and the
oracle, at the edges of the product kernel's tiles (64-lane strips of 256 / 512 / 1024 columns,
blocks of 8 selected rows, 8 wavefronts, shares)."""
import numpy as np
import pytest
import torch

from oracle import dip_oracle as O
from workloads import ar1_laplace_stream, layer_weights
from gpu_util import assert_product_close, dev_f32, host_u32, make_weight, rel_l2, workspace

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def D():
    import paper_2412_01380_amd as D
    return D


def _layers(D, dims, fmt):
    ws = [layer_weights(d, f, seed=71, layer=l, dtype=fmt) for l, (d, f) in enumerate(dims)]
    return ws, [D.Mlp(make_weight(D, w["ug"]), make_weight(D, w["d"])) for w in ws]


def _caches(D, dims, policy=0):
    cs = [[D.Cache(d, d // 2, policy) for d, _ in dims], [D.Cache(f, f // 2, policy) for _, f in dims]]
    for c in cs[0] + cs[1]:
        D.dip_cache_init(c)
    return cs


def _check(D, dims, fmt, k_in, k_mid, use_cache, tokens=3):
    """A stack call per token against per-layer calls on a second set of caches: y against the
    oracle's product of the per-layer call's h and mask, cache states bit for bit."""
    ws, mlps = _layers(D, dims, fmt)
    L, d = len(dims), dims[0][0]
    a, b = (_caches(D, dims), _caches(D, dims)) if use_cache else ((None, None), (None, None))
    stack = D.MlpStack(mlps, a[0], a[1])
    buf = workspace(D.dip_swiglu_mlp_forward_stack_workspace_bytes(stack, k_in, k_mid))
    buf.fill_(0xFF)       # nothing is expected of the workspace's contents
    one = workspace(max(D.dip_swiglu_mlp_forward_workspace_bytes(m, k_in[l], k_mid[l]) for l, m in enumerate(mlps)))
    X = dev_f32(ar1_laplace_stream(L * tokens, d, seed=72).reshape(tokens, L, d))
    Y = torch.full((L, d), float("nan"), device="cuda")
    y1 = torch.empty(d, device="cuda")
    for t in range(tokens):
        D.dip_swiglu_mlp_forward_stack(stack, X[t], d, k_in, k_mid, 0.2, Y, d, buf)
        for l, (_, f) in enumerate(dims):
            dbg = D.Debug(d, f, k_in[l], k_mid[l])
            D.dip_swiglu_mlp_forward(mlps[l], X[t, l], k_in[l], k_mid[l], b[0] and b[0][l], b[1] and b[1][l], 0.2, y1, dbg, one)
            torch.cuda.synchronize()
            ref = O.gathered_gemv(ws[l]["d"], dbg.h.cpu().numpy(), dbg.idx_mid.cpu().numpy())
            # h of the two calls differs by the rounding of its own sums (k_in terms, then SwiGLU)
            assert_product_close(Y[l].cpu().numpy(), ref, fmt, max(k_in[l], k_mid[l]), (t, l, "y"), factor=4.0)
            if use_cache:
                for p, q in ((a[0][l], b[0][l]), (a[1][l], b[1][l])):
                    assert torch.equal(p.bits, q.bits) and torch.equal(p.stamp, q.stamp) and torch.equal(p.meta, q.meta), (t, l)


@pytest.mark.parametrize("fmt,d,f", [("f32", 516, 1540), ("bf16", 520, 1544), ("bf16", 1032, 2056), ("int4", 640, 1408)])
def test_stack_edges_of_tiles_blocks_and_shares(D, fmt, d, f):
    # per-layer k: below, at and above one block and one round of blocks, a prime, everything
    k_in = [1, 7, 8, 9, 63, 64, 65, d - 1, d]
    k_mid = [d, 65, 64, 63, 9, 8, 7, 1, f]
    _check(D, [(d, f)] * 9, fmt, k_in, k_mid, use_cache=True)


def test_stack_of_runs_and_single_layers(D):
    """Phases for the runs, layer by layer in between: both share one scratch area."""
    dims = [(512, 1536)] * 4 + [(512, 2304)] + [(512, 1024)] * 5 + [(512, 1536)] * 2
    L = len(dims)
    _check(D, dims, "bf16", [150] * L, [400 + 8 * l for l in range(L)], use_cache=True)
    _check(D, dims, "f32", [150] * L, [400 + 8 * l for l in range(L)], use_cache=False)


def test_stack_longer_than_one_table(D):
    _check(D, [(256, 512)] * 70, "bf16", [80] * 70, [200] * 70, use_cache=True, tokens=2)


def test_stack_layers_chained_through_their_buffers(D):
    """y of layer l is x of layer l + 1: such a call runs its layers one after the other."""
    dims, k_in, k_mid = [(512, 1536)] * 5, 160, 500
    _, mlps = _layers(D, dims, "bf16")
    stack = D.MlpStack(mlps)
    buf = workspace(D.dip_swiglu_mlp_forward_stack_workspace_bytes(stack, k_in, k_mid))
    chain = torch.zeros(6, 512, device="cuda")
    chain[0] = dev_f32(ar1_laplace_stream(1, 512, seed=3)[0])
    want = chain.clone()
    D.dip_swiglu_mlp_forward_stack(stack, chain, 512, k_in, k_mid, 0.2, chain[1:], 512, buf)
    for l in range(5):
        D.dip_swiglu_mlp_forward(mlps[l], want[l], k_in, k_mid, None, None, 0.2, want[l + 1], None, buf)
    torch.cuda.synchronize()
    assert torch.equal(chain.view(torch.int32), want.view(torch.int32))
    # in place (y over its own x) keeps the phases
    x = dev_f32(ar1_laplace_stream(5, 512, seed=4))
    y = torch.empty_like(x)
    D.dip_swiglu_mlp_forward_stack(stack, x, 512, k_in, k_mid, 0.2, y, 512, buf)
    D.dip_swiglu_mlp_forward_stack(stack, x, 512, k_in, k_mid, 0.2, x, 512, buf)
    torch.cuda.synchronize()
    assert torch.equal(x.view(torch.int32), y.view(torch.int32))


def test_stack_of_non_finite_inputs_ends(D):
    dims = [(512, 1536)] * 4
    _, mlps = _layers(D, dims, "bf16")
    stack = D.MlpStack(mlps)
    buf = workspace(D.dip_swiglu_mlp_forward_stack_workspace_bytes(stack, 160, 500))
    buf.fill_(0xFF)
    x = torch.randn(4, 512, device="cuda")
    x[0, 3], x[1, ::2], x[2] = float("inf"), float("nan"), float("nan")
    y = torch.empty_like(x)
    D.dip_swiglu_mlp_forward_stack(stack, x, 512, 160, 500, 0.2, y, 512, buf)
    torch.cuda.synchronize()
    assert torch.isfinite(y[3]).all()


@pytest.mark.parametrize("fmt", ["bf16", "int4"])
def test_stack_phases_replay_from_a_graph(D, fmt):
    dims, k_in, k_mid, L = [(512, 1536)] * 6, 150, 500, 6
    _, mlps = _layers(D, dims, fmt)
    ce, cg = _caches(D, dims), _caches(D, dims)
    se, sg = D.MlpStack(mlps, *ce), D.MlpStack(mlps, *cg)
    n = D.dip_swiglu_mlp_forward_stack_workspace_bytes(se, k_in, k_mid)
    we, wg = workspace(n), workspace(n)
    X = dev_f32(ar1_laplace_stream(L * 5, 512, seed=8).reshape(5, L, 512))
    xb, ye, yg = torch.zeros(L, 512, device="cuda"), torch.empty(L, 512, device="cuda"), torch.zeros(L, 512, device="cuda")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        D.dip_swiglu_mlp_forward_stack(sg, xb, 512, k_in, k_mid, 0.2, yg, 512, wg)
    for t in range(5):
        D.dip_swiglu_mlp_forward_stack(se, X[t], 512, k_in, k_mid, 0.2, ye, 512, we)
        xb.copy_(X[t])
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(ye.view(torch.int32), yg.view(torch.int32)), t
        for a, b in zip(ce[0] + ce[1], cg[0] + cg[1]):
            assert np.array_equal(host_u32(a.bits), host_u32(b.bits)) and a.meta_host() == b.meta_host(), t


def _in_order(D, mlps, buf, x_at, x_stride, y_at, y_stride, B, d, k_in, k_mid):
    """The same call, layer by layer, on `buf`: one-row calls (B = 0) or batched ones."""
    one = workspace(max(D.dip_swiglu_mlp_forward_workspace_bytes(mlps[0], k_in, k_mid),
                        D.dip_swiglu_mlp_forward_batched_workspace_bytes(mlps[0], max(B, 1), k_in, k_mid)))
    for l, m in enumerate(mlps):
        x, y = buf[x_at + l * x_stride:], buf[y_at + l * y_stride:]
        if B == 0:
            D.dip_swiglu_mlp_forward(m, x, k_in, k_mid, None, None, 0.2, y, None, one)
        else:
            D.dip_swiglu_mlp_forward_batched(m, x, B, k_in, k_mid, None, None, 0.2, y, None, None, None, one)


@pytest.mark.parametrize("B", [0, 1, 3])
@pytest.mark.parametrize("case", ["one place", "half a row", "half a row down", "one short", "chained", "last row chained",
                                  "interleaved"])
def test_stack_layers_with_overlapping_rows_run_in_order(D, case, B):
    """Outputs that overlap each other or a later layer's inputs, through both stack calls (B = 0:
    the one-row call): the bits of one call per layer, in order."""
    d, f, L, k_in, k_mid = 512, 1536, 6, 160, 500
    rows = max(B, 1)
    R = rows * d                                         # floats a layer reads and writes
    x_at, x_stride, far = 0, R, (L + 1) * R
    y_at, y_stride = {
        "one place": (far, 0),
        "half a row": (far, d // 2),
        "half a row down": (far + L * R, -(d // 2)),
        "one short": (far, R - 1),                       # one float of the last batch row only
        "chained": (R, R),                               # y of layer l is x of layer l + 1
        "last row chained": (2 * R - (rows - 1) * d, 2 * R),
        "interleaved": (R, 2 * R),                       # [x0 y0 x1 y1 ...]: nothing overlaps
    }[case]
    if case in ("last row chained", "interleaved"):
        x_stride = 2 * R
    _, mlps = _layers(D, [(d, f)] * L, "bf16")
    stack = D.MlpStack(mlps)
    start = dev_f32(ar1_laplace_stream(1, 4 * (L + 1) * R, seed=12)[0])
    got, want = start.clone(), start.clone()
    if B == 0:
        ws = workspace(D.dip_swiglu_mlp_forward_stack_workspace_bytes(stack, k_in, k_mid))
        D.dip_swiglu_mlp_forward_stack(stack, got[x_at:], x_stride, k_in, k_mid, 0.2, got[y_at:], y_stride, ws)
    else:
        ws = workspace(D.dip_swiglu_mlp_forward_batched_stack_workspace_bytes(stack, B, k_in, k_mid))
        D.dip_swiglu_mlp_forward_batched_stack(stack, got[x_at:], x_stride, B, k_in, k_mid, 0.2, got[y_at:], y_stride, ws)
    _in_order(D, mlps, want, x_at, x_stride, y_at, y_stride, B, d, k_in, k_mid)
    torch.cuda.synchronize()
    if case == "interleaved":                            # runs in phases: the rounding of another split of the sums
        assert torch.allclose(got, want, rtol=0, atol=4e-6 * float(want.abs().max()))
    else:
        assert torch.equal(got.view(torch.int32), want.view(torch.int32))


@pytest.mark.parametrize("B", [0, 1, 2])
@pytest.mark.parametrize("scale_log2", [62, 0, -60])
def test_stack_int4_at_both_ends_of_the_fp32_range(D, B, scale_log2):
    """The int4 product of the stacks keeps its codes as fp16 denormals and moves their factor into
    multipliers and sums: the GLU outputs here reach 2^125 (largest) and 2^-122 (root mean square),
    where neither has room for a fixed factor.  Through both stack calls (B = 0: the one-row call)."""
    d, f, L, k_in, k_mid = 1152, 4224, 64, 400, 4100     # (a batch takes this kernel from so many rows on)
    (w,), (mlp,) = _layers(D, [(d, f)], "int4")
    stack = D.MlpStack([mlp] * L)
    R = max(B, 1)
    X = np.stack([ar1_laplace_stream(1, d, seed=400 + i)[0] for i in range(L * R)]).reshape(L, R, d)
    X[:, 0] *= np.float32(2.0 ** scale_log2)
    Y = torch.full((L, R, d), float("nan"), device="cuda")
    if B == 0:
        ws = workspace(D.dip_swiglu_mlp_forward_stack_workspace_bytes(stack, k_in, k_mid))
        D.dip_swiglu_mlp_forward_stack(stack, dev_f32(X), d, k_in, k_mid, 0.2, Y, d, ws)
    else:
        ws = workspace(D.dip_swiglu_mlp_forward_batched_stack_workspace_bytes(stack, B, k_in, k_mid))
        D.dip_swiglu_mlp_forward_batched_stack(stack, dev_f32(X), B * d, B, k_in, k_mid, 0.2, Y, B * d, ws)
    torch.cuda.synchronize()
    Yg = Y.cpu().numpy()
    for l in (0, L - 1):
        for b in range(R):
            _, idx1 = O.topk(O.score(X[l, b], None, 0.2), k_in)
            with np.errstate(over="ignore", under="ignore"):
                h = O.glu_from_preacts(O.gathered_gemv(w["ug"], X[l, b], idx1))
            assert np.all(np.isfinite(h)) and (b > 0 or scale_log2 != 62 or np.abs(h).max() > 2.0 ** 124)
            _, idx2 = O.topk(O.score(h, None, 0.2), k_mid)
            # (sums of 4100 terms round to a few 1e-7, at -60 with steps of 2^-149 on 2^-122)
            assert rel_l2(Yg[l, b], O.gathered_gemv(w["d"], h, idx2)) <= 4e-6, (l, b)


@pytest.mark.parametrize("fmt,B", [("f32", 0), ("f32", 2), ("bf16", 0), ("bf16", 2), ("bf16", 8), ("int4", 0), ("int4", 1),
                                   ("int4", 2)])
def test_stack_sums_are_as_exact_as_a_layer_on_its_own(D, fmt, B):
    """Error of y against 64 bits, through a stack call of 40 layers and through one call per layer (B = 0:
    the one-row calls).  The rounding of a sum grows with the square root of its longest chain: sums
    that run through a wavefront's whole share in one chain, 8 times the rows of a layer on its own,
    come out 1.17 to 2.7 times as far off.  Half of the columns kept; the median of 8 rows, each of
    2048 outputs, whose error norms agree to about 5 %."""
    d, f, L, k_in, k_mid = 2048, 6144, 40, 1024, 3072
    (w,), (mlp,) = _layers(D, [(d, f)], fmt)
    stack = D.MlpStack([mlp] * L)
    R = max(B, 1)
    X = np.stack([ar1_laplace_stream(1, d, seed=900 + i)[0] for i in range(L * R)]).reshape(L, R, d)
    Xd, Y, Y1 = dev_f32(X), torch.empty(L, R, d, device="cuda"), torch.empty(L, R, d, device="cuda")
    if B == 0:
        ws = workspace(D.dip_swiglu_mlp_forward_stack_workspace_bytes(stack, k_in, k_mid))
        D.dip_swiglu_mlp_forward_stack(stack, Xd, d, k_in, k_mid, 0.2, Y, d, ws)
        for l in range(L):
            D.dip_swiglu_mlp_forward(mlp, Xd[l], k_in, k_mid, None, None, 0.2, Y1[l], None, ws)
    else:
        ws = workspace(D.dip_swiglu_mlp_forward_batched_stack_workspace_bytes(stack, B, k_in, k_mid))
        D.dip_swiglu_mlp_forward_batched_stack(stack, Xd, B * d, B, k_in, k_mid, 0.2, Y, B * d, ws)
        for l in range(L):
            D.dip_swiglu_mlp_forward_batched(mlp, Xd[l], B, k_in, k_mid, None, None, 0.2, Y1[l], None, None, None, ws)
    torch.cuda.synchronize()
    errs = []
    for i in range(8):
        l, b = i * 5, i % R
        _, idx1 = O.topk(O.score(X[l, b], None, 0.2), k_in)
        u = O.gathered_gemv(w["ug"], X[l, b], idx1)
        h = u[:f] * O.silu(u[f:])                        # 64 bits
        idx2 = np.sort(np.argsort(-np.abs(h), kind="stable")[:k_mid])
        y = h[idx2] @ O.widen_rows(w["d"], idx2)
        errs.append([rel_l2(a[l, b].cpu().numpy(), y) for a in (Y, Y1)])
    stacked, single = np.median(np.array(errs), axis=0)
    assert stacked <= 1.15 * single, (stacked, single)
