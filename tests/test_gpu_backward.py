"""GPU parity of the fp32 backward (cyfa_backward, kernel VALU) against the
backward oracle (head dims 64 and 128 in any combination, and both 256).

Every gradient tensor is compared element by element with the oracle's float64
reverse-mode gradients on the same seeded inputs, the same upstream gradient
d_o and the same final-state adjoints.  Error per tensor: max |x - y| / max |y|.
Bars: 1e-4 for float32 inputs, 2e-2 for bfloat16 inputs (fp32 arithmetic).
"""
import numpy as np
import pytest

from oracle import backward as ob
from paper_2609_36259_amd.inputs import make_forward_inputs
from tests.harness import TOL_BF16, TOL_F32, rel_err, upload

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _cyfa():
    from paper_2609_36259_amd import cyfa
    return cyfa


def _round(a, dtype):
    if dtype != "bf16":
        return np.asarray(a, np.float32)
    return torch.tensor(np.asarray(a, np.float32)).bfloat16().float().numpy()


def _extras(x, seed, init=True, final=True):
    """Upstream gradient, initial states/clock and final-state adjoints."""
    B, T, H = x["delta"].shape
    dk, dv, m = x["q"].shape[-1], x["v"].shape[-1], x["m"]
    rng = np.random.default_rng(seed)
    e = {"do": _round(rng.standard_normal((B, T, H, dv)), x["dtype"])}
    if init:
        K0 = np.zeros((B, H, 128, dk), np.float32)
        V0 = np.zeros((B, H, 128, dv), np.float32)
        K0[:, :, :m] = 0.3 * rng.standard_normal((B, H, m, dk))
        V0[:, :, :m] = 0.3 * rng.standard_normal((B, H, m, dv))
        e.update(K0=K0, V0=V0, clock0=rng.uniform(0, 2 * m, (B, H)))
    if final:
        dK = np.zeros((B, H, 128, dk), np.float32)
        dV = np.zeros((B, H, 128, dv), np.float32)
        dK[:, :, :m] = rng.standard_normal((B, H, m, dk))
        dV[:, :, :m] = rng.standard_normal((B, H, m, dv))
        e.update(dK_T=dK, dV_T=dV)
    return e


def _run(x, e, lens=None, groups=0):
    """The fp32 backward; the bf16 matrix-core one has its own file."""
    cyfa = _cyfa()
    t = upload(x)
    dt = t["q"].dtype
    dev = lambda a, dtype=torch.float32: None if a is None else torch.tensor(a, dtype=dtype, device="cuda")  # noqa: E731
    g = cyfa.backward(t["q"], t["k"], t["v"], t["delta"], t["log_alpha"], t["beta"], t["R"],
                      d_o=dev(e["do"], dt), scale=x["scale"], m=x["m"],
                      K0=dev(e.get("K0")), V0=dev(e.get("V0")),
                      clock0=dev(e.get("clock0"), torch.float64),
                      dK_T=dev(e.get("dK_T")), dV_T=dev(e.get("dV_T")),
                      lens=None if lens is None else dev(lens, torch.int32), groups=groups,
                      kernel=cyfa.KERNEL_VALU)
    torch.cuda.synchronize()
    return {k: (None if v is None else v.float().cpu().numpy() if v.dtype != torch.float64
                else v.cpu().numpy()) for k, v in g.items()}


def _oracle(x, e, lens=None):
    return ob.backward(x["q"], x["k"], x["v"], x["delta"], x["log_alpha"], x["beta"], x["R"],
                       do=e["do"], m=x["m"], scale=x["scale"], K0=e.get("K0"), V0=e.get("V0"),
                       clock0=e.get("clock0"), dK_T=e.get("dK_T"), dV_T=e.get("dV_T"), lens=lens)


PAIRS = {"dq": "dq", "dk": "dk", "dv": "dv", "d_delta": "ddelta", "d_log_alpha": "dlog_alpha",
         "d_beta": "dbeta", "d_R": "dR", "d_K0": "dK0", "d_V0": "dV0", "d_clock0": "dclock0"}


def _compare(g, ref, tol, skip=()):
    errs = {}
    for gk, rk in PAIRS.items():
        if gk in skip or ref.get(rk) is None:
            continue
        assert g[gk] is not None, gk
        errs[gk] = rel_err(g[gk], ref[rk])
    print("errors", {k: f"{v:.2e}" for k, v in errs.items()}, flush=True)
    for k, v in errs.items():
        assert v <= tol, (k, v)
    return errs


@pytest.mark.parametrize("m", [7, 127])
def test_f32_d64_full_parity(m):
    x = make_forward_inputs(2, 45, 2, 64, 64, seed=71, dtype="f32", m=m)
    e = _extras(x, 1)
    _compare(_run(x, e), _oracle(x, e), TOL_F32)


@pytest.mark.parametrize("dk,dv", [(128, 128), (64, 128), (128, 64)])
def test_f32_head_dims(dk, dv):
    x = make_forward_inputs(1, 37, 2, dk, dv, seed=72, dtype="f32")
    e = _extras(x, 2)
    _compare(_run(x, e), _oracle(x, e), TOL_F32)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_head_dim_256(dtype):
    """The paper's head size (d_k = d_v = 256; its 400M model's layer), initial
    states, final-state adjoints, two chunk groups and a ragged tail."""
    x = make_forward_inputs(2, 16 * 3 + 5, 2, 256, 256, seed=79, dtype=dtype)
    e = _extras(x, 9)
    _compare(_run(x, e, groups=2), _oracle(x, e), TOL_F32 if dtype == "f32" else TOL_BF16)


def test_head_dim_256_ragged():
    T = 16 * 3 + 7
    x = make_forward_inputs(3, T, 1, 256, 256, seed=80, dtype="f32")
    e = _extras(x, 10)
    lens = [T, 20, 0]
    g = _run(x, e, lens=lens, groups=2)
    _compare(g, _oracle(x, e, lens=lens), TOL_F32)
    for name in ("dq", "dk", "dv", "d_delta"):
        assert np.all(g[name][1, 20:] == 0) and np.all(g[name][2] == 0), name


def test_bf16_d128():
    x = make_forward_inputs(2, 50, 2, 128, 128, seed=73, dtype="bf16")
    e = _extras(x, 3)
    _compare(_run(x, e), _oracle(x, e), TOL_BF16)


def test_absent_gates_readout_and_states():
    x = make_forward_inputs(1, 40, 2, 64, 64, seed=74, dtype="f32", with_beta=False, with_R=False)
    x["log_alpha"] = None
    e = _extras(x, 4, init=False, final=False)
    g = _run(x, e)
    assert g["d_log_alpha"] is None and g["d_beta"] is None and g["d_R"] is None
    _compare(g, _oracle(x, e), TOL_F32)


def test_ragged_lengths():
    x = make_forward_inputs(3, 40, 2, 64, 64, seed=75, dtype="f32")
    e = _extras(x, 5)
    lens = [40, 19, 0]
    g = _run(x, e, lens=lens)
    ref = _oracle(x, e, lens=lens)
    _compare(g, ref, TOL_F32)
    for name in ("dq", "dk", "dv", "d_delta", "d_log_alpha", "d_beta"):
        assert np.all(g[name][1, 19:] == 0) and np.all(g[name][2] == 0), name


def test_chunk_groups_change_only_rounding():
    x = make_forward_inputs(1, 16 * 7 + 3, 2, 64, 64, seed=76, dtype="f32")
    e = _extras(x, 6)
    a = _run(x, e, groups=1)
    b = _run(x, e, groups=3)
    for k in PAIRS:
        assert rel_err(b[k], a[k]) <= 1e-5, k


def test_peaky_logits():
    """A large logit scale makes the softmax far from uniform, so errors in the
    readout's adjoint are not hidden by near-constant weights."""
    x = make_forward_inputs(1, 33, 2, 64, 64, seed=77, dtype="f32")
    x["scale"] = 12.0
    e = _extras(x, 7)
    _compare(_run(x, e), _oracle(x, e), TOL_F32)


def test_empty_sequence_passes_state_adjoints_through():
    x = make_forward_inputs(1, 0, 2, 64, 64, seed=78, dtype="f32")
    e = _extras(x, 8)
    g = _run(x, e)
    np.testing.assert_array_equal(g["d_K0"], e["dK_T"])
    np.testing.assert_array_equal(g["d_V0"], e["dV_T"])
    assert np.all(g["d_clock0"] == 0)


@pytest.mark.timeout(400)
def test_full_size_sampled_sequence():
    """The 1.4B-scale workload (B=4, T=4096, H=16, d=128, bf16) in the launch
    configuration the benchmark times (automatic chunk groups); one sampled
    (b, h) sequence's gradients, all tokens, against the oracle run on that
    sequence alone (dR sums over every sequence and is covered by the small cases)."""
    from paper_2609_36259_amd.inputs import FWD_1P4B, workload_inputs
    x = workload_inputs(FWD_1P4B)
    B, T, H = x["delta"].shape
    rng = np.random.default_rng(9)
    e = {"do": _round(rng.standard_normal((B, T, H, 128)), "bf16")}
    print("full-size backward", flush=True)
    g = _run(x, e)
    b, h = 2, 11
    sl = lambda a: None if a is None else np.ascontiguousarray(a[b:b + 1, :, h:h + 1])  # noqa: E731
    y = dict(x, q=sl(x["q"]), k=sl(x["k"]), v=sl(x["v"]), delta=sl(x["delta"]),
             log_alpha=sl(x["log_alpha"]), beta=sl(x["beta"]), R=x["R"][h:h + 1])
    print("oracle on sequence", (b, h), flush=True)
    ref = _oracle(y, {"do": sl(e["do"])})
    pick = {k: (v[b:b + 1, :, h:h + 1] if k in ("dq", "dk", "dv", "d_delta", "d_log_alpha", "d_beta")
                else v[b:b + 1, h:h + 1] if k in ("d_K0", "d_V0", "d_clock0") else v)
            for k, v in g.items() if v is not None}
    _compare(pick, ref, TOL_BF16, skip=("d_R",))


@pytest.mark.parametrize("B,T,H,d,lens", [
    (1, 1, 1, 64, None),                      # one token
    (1, 63, 2, 64, None), (1, 64, 1, 128, None), (2, 65, 1, 64, (65, 31)),   # around one 64-token chunk
    (1, 129, 1, 256, None),                   # three chunks: the readout's last pair has one
    (8, 65, 4, 256, (65, 64, 33, 32, 31, 1, 0, 65)),   # 256 workgroups: states walked, not scanned
])
def test_f32_chunk_edges(B, T, H, d, lens):
    """Tile, chunk and chunk-pair edges, and both ways of forming the chunks' states.
    Bar 1e-4 as everywhere for fp32 (sums of up to 256 products: ~1e-6)."""
    x = make_forward_inputs(B, T, H, d, d, seed=90 + T, dtype="f32")
    e = _extras(x, 12)
    _compare(_run(x, e, lens=None if lens is None else np.array(lens, np.int32)),
             _oracle(x, e, lens=None if lens is None else np.array(lens, np.int32)), TOL_F32)


def test_f32_strong_decay():
    """Stretches of log alpha = -6 and -40 inside a chunk: decays are differences of
    prefix sums of up to 2560, which a float sum would give to 1e-4 only."""
    x = make_forward_inputs(1, 128, 2, 64, 64, seed=97, dtype="f32")
    x["log_alpha"][:, 10:40] = -6.0
    x["log_alpha"][:, 64:110] = -40.0
    e = _extras(x, 13)
    _compare(_run(x, e), _oracle(x, e), TOL_F32)


@pytest.mark.parametrize("H", [2, 200])
def test_f32_hard_resets(H):
    """Forget gates of the type's lowest value, two in one 64-token chunk (short and long calls'
    kernels): the tokens after a reset keep their own decays."""
    x = make_forward_inputs(1, 100, H, 64, 64, seed=98, dtype="f32")
    x["log_alpha"][:, [10, 30, 70]] = np.finfo(np.float32).min
    e = _extras(x, 17)
    _sampled(x, e, None, _run(x, e), 0, H - 1, TOL_F32)


def _sampled(x, e, lens, g, b, h, tol, skip=()):
    """One sequence of a batch against the oracle run on that sequence alone."""
    sl = lambda a: None if a is None else np.ascontiguousarray(a[b:b + 1, :, h:h + 1])  # noqa: E731
    ss = lambda a: None if a is None else np.ascontiguousarray(a[b:b + 1, h:h + 1])     # noqa: E731
    y = dict(x, q=sl(x["q"]), k=sl(x["k"]), v=sl(x["v"]), delta=sl(x["delta"]),
             log_alpha=sl(x["log_alpha"]), beta=sl(x["beta"]), R=x["R"][h:h + 1])
    f = dict({n: ss(e[n]) for n in e if n != "do"}, do=sl(e["do"]))
    ref = _oracle(y, f, lens=None if lens is None else lens[b:b + 1])
    pick = {k: (v[b:b + 1, :, h:h + 1] if k in ("dq", "dk", "dv", "d_delta", "d_log_alpha", "d_beta")
                else v[b:b + 1, h:h + 1] if k in ("d_K0", "d_V0", "d_clock0") else v[h:h + 1])
            for k, v in g.items() if v is not None}
    _compare(pick, ref, tol, skip=skip)


@pytest.mark.parametrize("B,T,H,dk,dv,m,dtype,lens", [
    (1, 129, 86, 64, 64, 127, "f32", None),        # 258 chunks; the last pair of a sequence has one
    (1, 128, 129, 64, 128, 31, "f32", None),
    (2, 129, 43, 128, 64, 127, "f32", (129, 66)),
    (2, 65, 65, 128, 128, 127, "f32", (65, 1)),      # (0: the clock gradient is 0, the oracle's its rounding)
    (1, 129, 86, 64, 64, 127, "bf16", None),
])
def test_long_call_kernels(B, T, H, dk, dv, m, dtype, lens):
    """Calls just over 256 chunks, at chunk-pair edges: first, middle and last sequence (with
    one batch entry d_R is the sequence's own)."""
    x = make_forward_inputs(B, T, H, dk, dv, seed=140 + T, dtype=dtype, m=m)
    e = _extras(x, 14)
    lens = None if lens is None else np.array(lens, np.int32)
    g = _run(x, e, lens=lens)
    for b, h in ((0, 0), (0, H // 2), (B - 1, H - 1)):
        _sampled(x, e, lens, g, b, h, TOL_F32 if dtype == "f32" else TOL_BF16, skip=() if B == 1 else ("d_R",))


@pytest.mark.parametrize("B,T,H,dk,dv,m,dtype", [
    (1, 32, 2, 64, 128, 127, "f32"), (3, 33, 1, 128, 64, 3, "f32"), (2, 96, 2, 128, 128, 65, "f32"),
    (1, 97, 1, 64, 64, 127, "bf16"), (1, 200, 64, 64, 64, 127, "f32"),     # 256 chunks: the line
])
def test_short_call_tile_edges(B, T, H, dk, dv, m, dtype):
    """32-token tile edges of the short calls' kernels, their head dimensions and small m."""
    x = make_forward_inputs(B, T, H, dk, dv, seed=150 + T, dtype=dtype, m=m)
    e = _extras(x, 15)
    g = _run(x, e)
    for b, h in {(0, 0), (B - 1, H - 1)}:
        _sampled(x, e, None, g, b, h, TOL_F32 if dtype == "f32" else TOL_BF16, skip=() if B == 1 else ("d_R",))


def test_short_call_many_sequences_share_workgroups():
    """600 sequences of up to two tiles: more tiles than the readout kernel has workgroups, whose
    dM then sums several tiles, absent ones among them.  Against the same sequences 150 at a
    time, one tile per workgroup: the token gradients bit for bit, d_R to 1e-5 (fp32 sums of
    the same terms in another order)."""
    cyfa = _cyfa()
    B, T, H, d = 600, 40, 1, 64
    g = torch.Generator(device="cuda")
    g.manual_seed(16)
    q, k, v, d_o = (torch.randn((B, T, H, d), device="cuda", generator=g) for _ in range(4))
    la, delta = -torch.rand((B, T, H), device="cuda", generator=g), torch.rand((B, T, H), device="cuda", generator=g)
    beta, R = torch.rand((B, T, H), device="cuda", generator=g), torch.eye(127, device="cuda")[None].contiguous()
    lens = torch.tensor([(40, 33, 32, 5, 0)[b % 5] for b in range(B)], dtype=torch.int32, device="cuda")
    run = lambda s: cyfa.backward(q[s], k[s], v[s], delta[s], la[s], beta[s], R, d_o=d_o[s], lens=lens[s])  # noqa: E731
    full, parts = run(slice(None)), [run(slice(i, i + 150)) for i in range(0, B, 150)]
    for name in ("dq", "dk", "dv", "d_delta", "d_log_alpha", "d_beta"):
        assert torch.equal(full[name], torch.cat([x[name] for x in parts])), name
    ref = sum(x["d_R"] for x in parts)
    assert (full["d_R"] - ref).abs().max() <= 1e-5 * ref.abs().max()
