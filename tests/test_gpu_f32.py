"""The float32 kernels at the edges of their tiles (64 slots, 64 columns, 32 k;
16 tokens of the router), against the oracle."""
import numpy as np
import pytest
import torch

from oracle import oracle
from paper_2601_05296_amd import binding as B
from tests.parity import assert_close, dev, host, near_tie_ok

pytestmark = pytest.mark.gpu


def _route(x, wg, bias, k, renorm):
    T, d = x.shape
    E = wg.shape[0]
    ids = torch.empty((T, k), dtype=torch.int32, device="cuda")
    gates = torch.empty((T, k), dtype=torch.float32, device="cuda")
    logits = torch.empty((T, E), dtype=torch.float32, device="cuda")
    B.moe_route(dev(x), dev(wg), dev(bias), T, d, E, k,
                B.MOE_F32 | (B.MOE_RENORM if renorm else 0), ids, gates, logits)
    torch.cuda.synchronize()
    return ids.cpu().numpy(), host(gates), host(logits)


@pytest.mark.parametrize("T,d,E,k,renorm", [
    (1, 64, 1, 1, False), (15, 64, 16, 16, True), (16, 128, 17, 3, False), (33, 192, 64, 8, True),
    (50, 64, 65, 5, False), (100, 320, 256, 16, True)])
def test_route_f32_edges(T, d, E, k, renorm):
    rng = np.random.Generator(np.random.PCG64(T + E))
    x = rng.standard_normal((T, d), dtype=np.float32)
    wg = rng.standard_normal((E, d), dtype=np.float32) * np.float32(0.02)
    bias = rng.standard_normal(E, dtype=np.float32)
    ids_r, gates_r, logits_r, _ = oracle.route(x, wg, bias, k, renorm)
    ids, gates, logits = _route(x, wg, bias, k, renorm)
    assert_close("logits", logits, logits_r, "f32")
    assert near_tie_ok(ids, ids_r, logits_r) <= 1
    same = np.all(ids == ids_r, axis=1)
    assert_close("gates", gates[same], gates_r[same], "f32")


def test_route_f32_ties_and_nan():
    """Equal logits go to the lower id; a NaN logit is never larger than a
    number, and is taken where it stands at the lowest free expert (so that the
    ids stay distinct and in range whatever the logits hold)."""
    E, k, T, d = 40, 6, 20, 64
    x = np.zeros((T, d), dtype=np.float32)      # every logit is its bias: ties
    bias = np.zeros(E, dtype=np.float32)
    bias[[7, 30]] = 1.0
    wg = np.zeros((E, d), dtype=np.float32)
    x[3] = np.nan                               # all logits of token 3 NaN
    bias2 = bias.copy()
    bias2[[0, 5]] = np.nan                      # two experts NaN for every token
    for b in (bias, bias2):
        ids, _, _ = _route(x, wg, b, k, False)
        for t in range(T):
            l = np.full(E, np.nan, np.float32) if t == 3 else b
            free, want = list(range(E)), []
            for _ in range(k):
                best = free[0]
                for e in free[1:]:
                    if l[e] > l[best]:
                        best = e
                want.append(best)
                free.remove(best)
            assert ids[t].tolist() == want, (t, want)


@pytest.mark.parametrize("counts,d,f,act", [
    ([1, 31, 63, 64, 65, 0, 128, 129], 64, 128, "swiglu"),
    ([33, 32, 95, 1], 192, 64, "silu"),
    ([66, 64], 64, 4224, "swiglu"),        # more column tiles than gate-gradient parts
    ([0, 70, 0], 128, 192, "relu")])
def test_ffn_f32_edges(counts, d, f, act):
    E, T, k = len(counts), sum(counts), 1
    rng = np.random.Generator(np.random.PCG64(T + f))
    ids = rng.permutation(np.repeat(np.arange(E), counts)).astype(np.int32)[:, None]

    def n(shape, s):
        return rng.standard_normal(shape, dtype=np.float32) * np.float32(s)

    x, dy, g = n((T, d), 1), n((T, d), 1), rng.random((T, 1), dtype=np.float32)
    w1, w3, w2 = n((E, d, f), d ** -0.5), n((E, d, f), d ** -0.5), n((E, f, d), f ** -0.5)
    gated = act == "swiglu"
    ix = oracle.build_index(ids, E)
    if gated:
        A_r, B_r, O_r = oracle.ffn_fwd(x, w1, w3, w2, ix, k)
        bw = oracle.ffn_bwd(dy, x, w1, w3, w2, g, ix, A_r, B_r)
    else:
        A_r, O_r = oracle.ffn_fwd_act(x, w1, w2, ix, k, act)
        bw = oracle.ffn_bwd_act(dy, x, w1, w2, g, ix, A_r, act)
    f32 = dict(dtype=torch.float32, device="cuda")
    A, O, dX = torch.empty((T, f), **f32), torch.empty((T, d), **f32), torch.empty((T, d), **f32)
    Bm = torch.empty((T, f), **f32) if gated else None
    base = n((E, d, f), 1)                        # dw1 is added to, as are dw3 and dw2
    dw1, dw2 = dev(base), dev(base.reshape(E, f, d))
    dw3 = dev(base) if gated else None
    dg = torch.empty((T, 1), **f32)
    fl = B.MOE_F32 | B.ACT_FLAG[act]
    xs, dys, w1s, w2s = dev(x), dev(dy), dev(w1), dev(w2)
    w3s = dev(w3) if gated else None
    off, eti, ss = dev(ix.offsets), dev(ix.eti), dev(ix.slot_src)
    B.moe_ffn_fwd(xs, w1s, w3s, w2s, off, eti, T, d, f, E, k, fl, A, Bm, O, None, 0)
    torch.cuda.synchronize()
    assert_close("A", host(A), A_r, "f32")
    assert_close("O", host(O), O_r, "f32")
    B.moe_ffn_bwd(dys, xs, w1s, w3s, w2s, dev(g), off, eti, ss, A, Bm, T, d, f, E, k,
                  fl | B.MOE_ACCUMULATE_DW, dw1, dw3, dw2, dg, dX, None, 0)
    torch.cuda.synchronize()
    assert_close("dA", host(A), bw["dA"], "f32")
    assert_close("dX_slot", host(dX), bw["dX_slot"], "f32")
    assert_close("d_gates", host(dg), bw["d_gates"], "f32")
    assert_close("dw1", host(dw1), bw["dw1"] + base, "f32")
    assert_close("dw2", host(dw2), bw["dw2"] + base.reshape(E, f, d), "f32")
    if gated:
        assert_close("dB", host(Bm), bw["dB"], "f32")
        assert_close("dw3", host(dw3), bw["dw3"] + base, "f32")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("over", ["dy", "x"])
def test_dX_slot_in_place_of_an_input(dtype, over):
    """Top-1: dX_slot [T, d] may take the place of dy or of x, which the backward has
    finished with when it writes dX_slot."""
    E, T, k, d, f = 5, 300, 1, 192, 320
    gen = torch.Generator(device="cuda").manual_seed(1)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16

    def n(*shape):
        return torch.randn(shape, generator=gen, device="cuda").mul_(shape[-1] ** -0.5).to(dt)

    ids = np.random.Generator(np.random.PCG64(1)).integers(0, E, (T, 1)).astype(np.int32)
    ix = oracle.build_index(ids, E)
    off, eti, ss = dev(ix.offsets), dev(ix.eti), dev(ix.slot_src)
    x, dy, A0, B0 = n(T, d), n(T, d), n(T, f), n(T, f)
    w1, w3, w2 = n(E, d, f), n(E, d, f), n(E, f, d)
    g = torch.rand((T, 1), generator=gen, device="cuda")
    fl = B.MOE_F32 if dtype == "f32" else 0
    nws = B.moe_ffn_bwd_workspace_size(T, d, f, E, k, fl)
    ws = torch.empty(max(nws, 16), dtype=torch.uint8, device="cuda")

    def run(in_place):
        f32 = dict(dtype=torch.float32, device="cuda")
        o = dict(A=A0.clone(), B=B0.clone(), dw1=torch.empty((E, d, f), **f32),
                 dw3=torch.empty((E, d, f), **f32), dw2=torch.empty((E, f, d), **f32),
                 dg=torch.empty((T, 1), **f32))
        xi, dyi = x.clone(), dy.clone()
        o["dX"] = {"dy": dyi, "x": xi}[over] if in_place else torch.empty((T, d), dtype=dt, device="cuda")
        B.moe_ffn_bwd(dyi, xi, w1, w3, w2, g, off, eti, ss, o["A"], o["B"], T, d, f, E, k, fl,
                      o["dw1"], o["dw3"], o["dw2"], o["dg"], o["dX"], ws, nws)
        torch.cuda.synchronize()
        return o

    apart, here = run(False), run(True)
    # float32 adds the gate gradient's column tiles in another order
    assert_close("d_gates", host(here.pop("dg")), host(apart.pop("dg")), "f32")
    for name, t in apart.items():
        assert torch.equal(t, here[name]), name
