"""The temporal attention, both directions, against a float64 evaluation at the edges of its kernels' sizes.

Widths that are one and several column groups, padded heads (head width not a multiple of 4), padded and
odd edge features, one and many slots (more than a half-wave's 32, a full wave's 64), 16- and 32-row blocks with
ragged ends, queries without slots and with a gap in their slots, rows at unaligned addresses, time
arguments past the fast range of the encoding, and dims that the general path takes, each of its kernels.
Gate: 1e-4 of each tensor's largest value in float32 (sums of at most a few hundred products: about
1e-6), 2e-2 in bfloat16 (a stored value that rounds the other way moves by 2^-8).
"""

import math

import numpy as np
import pytest
import torch

from paper_2608_16305_amd import mtgnn as M
from tests._gpu import log, needs_gpu, rel_err

pytestmark = [pytest.mark.gpu, needs_gpu]

NAMES = ("W_q", "W_k", "W_v", "W_o", "W_1", "W_2", "b_q", "b_k", "b_v", "b_o", "b_1", "b_2")


def _rnd(x, bf16):
    return x + (x.detach().float().bfloat16().double() - x.detach()) if bf16 else x


def _reference(p, mem, x, q_node, q_t, nbr, nt, neid, tw, tb, dz, H, bf16, uniq):
    """float64 on the CPU: z, the gradients and d_mem."""
    q64 = {n: v.double().requires_grad_() for n, v in p.items()}
    on = np.cumprod(nbr.numpy() >= 0, axis=1).astype(bool)
    on = torch.from_numpy(on)
    k, da = nbr.shape[1], p["W_q"].shape[0]
    m64 = mem.double().requires_grad_()
    w64, b64 = tw.double().requires_grad_(), tb.double().requires_grad_()

    def phi(dt):
        arg32 = tw * dt[..., None]
        arg32 = arg32 + tb
        arg = w64 * dt[..., None].double() + b64
        return _rnd(torch.cos(arg + (arg32.double() - arg).detach()), bf16)

    lin = lambda v, n: v @ q64["W_" + n].T + q64["b_" + n]   # noqa: E731
    Q = q_node.numel()
    hq = m64[q_node.long()]
    q = lin(torch.cat([hq, phi(torch.zeros(Q))], 1), "q").view(Q, 1, H, da // H)
    kv = [m64[nbr.clamp(min=0).long()]]
    if x is not None:
        kv.append(_rnd(x[neid.clamp(min=0).long()].double(), bf16))
    kv = torch.cat(kv + [phi(torch.where(on, q_t[:, None] - nt, torch.zeros(())))], 2)
    K, V = lin(kv, "k").view(Q, k, H, -1), lin(kv, "v").view(Q, k, H, -1)
    s = ((q * K).sum(3) / math.sqrt(da // H)).masked_fill(~on[..., None], -1e300)
    e = torch.exp(s - s.detach().amax(1, keepdim=True)) * on[..., None]
    a = ((e / e.sum(1, keepdim=True).clamp(min=1e-300))[..., None] * V).sum(1).reshape(Q, da)
    o = _rnd(lin(_rnd(a, bf16), "o"), bf16)
    z = lin(_rnd(torch.relu(lin(torch.cat([o, hq], 1), "1")), bf16), "2")
    z.backward(dz.double())
    g = {n: q64[n].grad.numpy() for n in NAMES}
    g.update(time_w=w64.grad.numpy(), time_b=b64.grad.numpy(), d_mem=m64.grad[uniq.long()].numpy())
    return z.detach().numpy(), g


#        H   dm   dt   de   da   k  max_q  n_q  dtype unaligned span
CASES = [(1, 4, 4, 0, 4, 1, 5, 5, "f32", False, 10.0),
         (2, 12, 8, 1, 12, 3, 33, 31, "f32", True, 1e5),
         (2, 100, 100, 3, 100, 20, 70, 66, "f32", False, 1e5),
         (1, 128, 128, 190, 128, 7, 40, 40, "f32", True, 1e3),
         (2, 128, 64, 256, 128, 64, 17, 17, "f32", False, 5e7),
         (2, 36, 100, 16, 20, 33, 48, 47, "f32", False, 1e4),
         (1, 32, 32, 2, 32, 5, 16_500, 16_400, "f32", True, 1e5),
         (2, 100, 100, 4, 100, 10, 16_400, 16_390, "f32", False, 1e5),
         (2, 64, 64, 172, 64, 9, 50, 49, "f32", False, 1e5),
         (2, 100, 100, 100, 100, 10, 33, 33, "f32", False, 1e5),
         (2, 20, 12, 29, 36, 8, 40, 37, "f32", True, 1e4),        # edge columns inside one tile of 16
         (1, 128, 128, 132, 128, 6, 33, 32, "bf16", False, 1e5),
         (2, 100, 100, 101, 100, 10, 37, 36, "bf16", True, 1e5),
         (2, 100, 100, 172, 100, 10, 20, 20, "bf16", False, 1e5),
         (2, 100, 100, 0, 100, 20, 50, 50, "bf16", False, 1e5),
         (1, 32, 32, 5, 32, 4, 35, 33, "bf16", True, 1e6),
         (4, 100, 100, 6, 100, 9, 45, 44, "f32", False, 1e4),      # general path: four heads
         (2, 30, 14, 3, 22, 6, 40, 39, "f32", False, 1e3),         # odd widths
         # the kernels for 16-byte groups: gather, key/value product and weight gradient of 200 columns by 200 and 216
         # (one row tile and many), softmax of up to 10 and 20 slots
         (4, 100, 100, 0, 100, 9, 45, 44, "f32", False, 1e4),
         (4, 100, 100, 16, 100, 12, 45, 44, "f32", False, 1e4),
         (4, 100, 100, 16, 100, 10, 3000, 2900, "f32", False, 1e4),
         (4, 100, 100, 0, 100, 9, 45, 44, "bf16", False, 1e4),
         (4, 100, 100, 16, 100, 10, 3000, 2900, "bf16", False, 1e4),
         (4, 36, 20, 5, 48, 7, 45, 44, "bf16", True, 1e4),
         (4, 100, 100, 0, 100, 1, 56_000, 55_990, "f32", False, 1e3),   # W_1's 200 columns: two groups, segments
         (2, 100, 100, 260, 100, 20, 45, 44, "f32", False, 1e4),
         (2, 100, 100, 260, 100, 9, 45, 44, "bf16", False, 1e4),
         (1, 96, 100, 260, 100, 20, 45, 44, "f32", False, 1e4),
         (1, 96, 100, 260, 100, 10, 45, 44, "f32", True, 1e4),
         (1, 160, 100, 8, 128, 30, 45, 44, "f32", False, 1e4),     # more than 20 slots, a head of 128
         # rows past 128 and 256 columns with few slots, to either side of the rule
         (2, 100, 100, 172, 100, 3, 45, 44, "f32", False, 1e4),
         (2, 100, 100, 172, 100, 4, 45, 44, "f32", False, 1e4),
         (2, 100, 100, 64, 100, 1, 45, 44, "f32", False, 1e4),
         (2, 100, 100, 64, 100, 2, 45, 44, "f32", False, 1e4),
         (1, 128, 128, 190, 128, 1, 45, 44, "bf16", False, 1e4)]


@pytest.mark.parametrize("H,dm,dt,de,da,k,max_q,n_q,dtype,unaligned,span", CASES)
def test_attention_sizes(H, dm, dt, de, da, k, max_q, n_q, dtype, unaligned, span):
    bf16 = dtype == "bf16"
    rng = np.random.default_rng(H * 1000 + dm * 7 + de * 3 + k)
    N, E = 97, 211
    store = torch.bfloat16 if bf16 else torch.float32
    log(f"[attn] H {H} dm {dm} dt {dt} de {de} da {da} k {k} queries {n_q}/{max_q} {dtype}")
    u = lambda *s: torch.from_numpy(rng.uniform(-1, 1, s).astype(np.float32))   # noqa: E731
    kv = dm + de + dt
    shapes = dict(W_q=(da, dm + dt), W_k=(da, kv), W_v=(da, kv), W_o=(da, da), W_1=(da, da + dm), W_2=(da, da))
    p = {}
    for n, (o, i) in shapes.items():
        p[n] = (u(o, i) * math.sqrt(6.0 / (o + i))).to(store)
        p["b" + n[1:]] = u(o) * 0.1
    tw = torch.from_numpy((10.0 ** (-6.0 * np.arange(dt) / max(dt - 1, 1))).astype(np.float32))
    tb = u(dt)
    mem, x = u(N, dm).to(store), (u(E, de) if de else None)
    q_node = torch.from_numpy(rng.integers(0, N, max_q).astype(np.int32))
    cnt = rng.integers(0, k + 1, max_q)
    nbr = rng.integers(0, N, (max_q, k)).astype(np.int32)
    nbr[np.arange(k)[None] >= cnt[:, None]] = -1
    gap = rng.random(max_q) < 0.1
    nbr[gap, k // 2] = -1   # slots behind a gap do not count
    nbr = torch.from_numpy(nbr)
    neid = torch.from_numpy(rng.integers(0, E, (max_q, k)).astype(np.int32))
    q_t = torch.from_numpy((span * (1 + rng.random(max_q))).astype(np.float32))
    nt = torch.from_numpy((span * rng.random((max_q, k))).astype(np.float32))
    dz = u(max_q, da) / max_q
    uniq = torch.from_numpy(rng.permutation(N)[:60].astype(np.int32))
    n_rows = 57
    z_ref, g_ref = _reference(p, mem, x, q_node[:n_q], q_t[:n_q], nbr[:n_q], nt[:n_q], neid[:n_q], tw, tb, dz[:n_q], H,
                              bf16, uniq[:n_rows])

    def dev(t, shift=False):
        if t is None:
            return None
        if not shift:
            return t.cuda()
        flat = torch.zeros(t.numel() + 1, dtype=t.dtype, device="cuda")
        flat[1:] = t.reshape(-1)
        return flat[1:].view(t.shape)

    pd = {n: dev(v) for n, v in p.items()}
    d = M.dims(N, dm, dt, de, da, H, k, M.BF16 if bf16 else M.F32)
    c_q, c_r = (torch.tensor([n], dtype=torch.int32, device="cuda") for n in (n_q, n_rows))
    nan = lambda *s: torch.full(s, math.nan, device="cuda")   # noqa: E731
    z, d_mem = nan(max_q, da), nan(60, dm)
    g = {n: nan(*p[n].shape) for n in NAMES}
    g.update(time_w=nan(dt), time_b=nan(dt))
    save = M.alloc_bytes(M.save_bytes(M.OP_TEMPORAL_ATTN, d, 0, max_q)).fill_(255)
    ws = M.alloc_bytes(max(M.workspace_bytes(M.OP_TEMPORAL_ATTN, d, 0, max_q),
                           M.workspace_bytes(M.OP_TEMPORAL_ATTN_BWD, d, 60, max_q))).fill_(255)
    args = [dev(t) for t in (q_node, q_t)] + [c_q, max_q] + [dev(t) for t in (nbr, nt)]
    td = dev(tw), dev(tb)
    M.mtgnn_temporal_attn(*args, dev(neid), dev(mem, unaligned), dev(x, unaligned), *td, M.attn_params(pd, d), d, z, save, ws)
    M.mtgnn_temporal_attn_bwd(*args, dev(dz, unaligned), save, dev(uniq), c_r, 60, *td, M.attn_params(pd, d), d,
                              M.attn_grads(g), d_mem, g["time_w"], g["time_b"], ws)
    torch.cuda.synchronize()
    errs = {"z": rel_err(z[:n_q].cpu().numpy(), z_ref)}
    g["d_mem"] = d_mem[:n_rows]
    for n, r in g_ref.items():
        got = g[n].cpu().numpy()
        if n == "b_k" or (n == "W_k" and k == 1):   # one slot: no score gradient but rounding
            errs[n] = float(np.abs(got).max() / np.abs(g_ref["W_v"]).max())
        elif n in ("W_q", "b_q") and k == 1:
            errs[n] = float(np.abs(got).max() / np.abs(g_ref["W_v"]).max())
        else:
            errs[n] = rel_err(got, r)
    log("  errors: " + ", ".join(f"{n}={v:.1e}" for n, v in errs.items()))
    assert all(math.isfinite(v) for v in errs.values()), errs
    assert max(errs.values()) <= (2e-2 if bf16 else 1e-4), errs
    assert torch.isnan(z[n_q:]).all()   # rows beyond the device count are left alone


def _forward_backward(p, mem, x, q_node, q_t, nbr, nt, neid, tw, tb, dz, H, k, uniq, bf16=False):
    """Both calls on the GPU: z, the gradients and d_mem on the CPU (every query and row counts)."""
    da, dm, dt = p["W_q"].shape[0], mem.shape[1], tw.numel()
    de = 0 if x is None else x.shape[1]
    d = M.dims(mem.shape[0], dm, dt, de, da, H, k, M.BF16 if bf16 else M.F32)
    Q, R = q_node.numel(), uniq.numel()
    c = lambda t: None if t is None else t.cuda()   # noqa: E731
    pd = {n: c(v) for n, v in p.items()}
    ap = M.attn_params(pd, d)
    c_q, c_r = (torch.tensor([n], dtype=torch.int32, device="cuda") for n in (Q, R))
    zero = lambda *s: torch.zeros(*s, device="cuda")   # noqa: E731
    z, d_mem = zero(Q, da), zero(R, dm)
    g = {n: zero(*p[n].shape) for n in NAMES}
    g.update(time_w=zero(dt), time_b=zero(dt))
    save = M.alloc_bytes(M.save_bytes(M.OP_TEMPORAL_ATTN, d, 0, Q))
    ws = M.alloc_bytes(max(M.workspace_bytes(M.OP_TEMPORAL_ATTN, d, 0, Q),
                           M.workspace_bytes(M.OP_TEMPORAL_ATTN_BWD, d, R, Q)))
    args = [c(q_node), c(q_t), c_q, Q, c(nbr), c(nt)]
    td = c(tw), c(tb)
    M.mtgnn_temporal_attn(*args, c(neid), c(mem), c(x), *td, ap, d, z, save, ws)
    M.mtgnn_temporal_attn_bwd(*args, c(dz), save, c(uniq), c_r, R, *td, ap, d, M.attn_grads(g), d_mem, g["time_w"],
                              g["time_b"], ws)
    torch.cuda.synchronize()
    return z.cpu(), {n: v.cpu() for n, v in g.items()}, d_mem.cpu()


def _passing(dm, dt, da):
    """Parameters of an embedding that hands its value sum's first da / 2 columns through exactly: z = relu(a) -
    relu(-a) there (d_mem and d_time columns of the values chosen by the caller in W_v)."""
    p = {n: torch.zeros(*s) for n, s in dict(W_q=(da, dm + dt), W_k=(da, dm + dt), W_v=(da, dm + dt), W_o=(da, da),
                                             W_1=(da, da + dm), W_2=(da, da)).items()}
    p.update({"b" + n[1:]: torch.zeros(da) for n in list(p)})
    h, i = da // 2, torch.arange(da // 2)
    p["W_o"].fill_diagonal_(1.0)
    p["W_1"][i, i], p["W_1"][h + i, i] = 1.0, -1.0
    p["W_2"][i, i], p["W_2"][i, h + i] = 1.0, -1.0
    return p


@pytest.mark.parametrize("span", [1.0, 100.0, 1e5, 1e6, 1e8])
def test_time_encoding_error(span):
    """The slots' cos(w dt + b) and, through b's gradient, its sine against 64 bits, the argument's product and sum
    rounded to float32.  Largest error 7.5e-8: half an ulp of the result (3.0e-8), half one of an argument of up to
    pi / 4 (3.0e-8 times a slope of 0.71 where it counts), 2.4e-8 for the polynomial and its sums; root mean
    square 1.8e-8, what the library's functions show."""
    dm, dt, da, Q = 4, 64, 128, 400
    log(f"[attn] time encoding, arguments to {span:g}")
    rng = np.random.default_rng(int(span))
    p = _passing(dm, dt, da)
    i = torch.arange(dt)
    p["W_v"][i, dm + i] = 1.0
    tw = torch.from_numpy((0.5 + 0.5 * rng.random(dt)).astype(np.float32))
    tb = torch.from_numpy(rng.uniform(-1, 1, dt).astype(np.float32))
    q_t = torch.from_numpy(rng.uniform(-span, span, Q).astype(np.float32))
    one = lambda v, t: torch.full((Q, 1), v, dtype=t)   # noqa: E731
    args = (torch.zeros(2, dm), None)
    arg = (tw * q_t[:, None]) + tb
    c64, s64 = torch.cos(arg.double()), torch.sin(arg.double())
    z, _, _ = _forward_backward(p, *args, torch.zeros(Q, dtype=torch.int32), q_t, one(1, torch.int32),
                                one(0.0, torch.float32), one(0, torch.int32), tw, tb, torch.zeros(Q, da), 1, 1,
                                torch.zeros(1, dtype=torch.int32))
    errs = [(z[:, :dt].double() - c64).numpy()]
    sines = []
    dz = torch.zeros(1, da)
    dz[0, :dt] = 1.0
    # relu passes one side: the slope of z in a is 1 either way (0 at a = 0)
    for r in range(0, Q, 8):
        _, g, _ = _forward_backward(p, *args, torch.zeros(1, dtype=torch.int32), q_t[r:r + 1], one(1, torch.int32)[:1],
                                    one(0.0, torch.float32)[:1], one(0, torch.int32)[:1], tw, tb, dz, 1, 1,
                                    torch.zeros(1, dtype=torch.int32))
        sines.append((-g["time_b"].double() - s64[r]).numpy())
    errs.append(np.stack(sines))
    for name, e in zip(("cos", "sin"), errs):
        log(f"  {name}: largest {np.abs(e).max():.2e}, rms {np.sqrt((e ** 2).mean()):.2e}")
    assert max(np.abs(e).max() for e in errs) <= 7.5e-8
    assert max(np.sqrt((e ** 2).mean()) for e in errs) <= 1.8e-8


@pytest.mark.parametrize("H,dtype", [(2, "f32"), (4, "f32"), (2, "bf16")])   # four heads: the general path
@pytest.mark.parametrize("Q", [3, 700, 20_000])
@pytest.mark.parametrize("kind", ["both", "largest", "infinite"])
def test_gradients_at_the_ends_of_the_range(H, dtype, Q, kind):
    """Infinite and nearly infinite output gradients: W_2's and b_2's gradients (a1 = 0.5 everywhere), and b_1's where
    W_2 does not turn them to NaN (0 times infinity), are the products float32 gives, infinite where it does and
    finite where it does, and the others' columns are what they are without them."""
    bf16 = dtype == "bf16"
    dm, da, k = 4, 100, 1
    big = float(np.finfo(np.float32).max)
    ends = {"both": {3: math.inf, 20: -math.inf, 41: big, 97: -big}, "largest": {41: big, 97: -big},
            "infinite": {20: -math.inf}}[kind]
    log(f"[attn] gradients at the ends of the range: H {H} {dtype} queries {Q} {kind}")
    rng = np.random.default_rng(H + Q)
    p = {n: torch.zeros(*s) for n, s in dict(W_q=(da, 2 * dm), W_k=(da, 2 * dm), W_v=(da, 2 * dm), W_o=(da, da),
                                             W_1=(da, da + dm), W_2=(da, da)).items()}
    p.update({"b" + n[1:]: torch.zeros(da) for n in list(p)})
    p["b_1"] += 0.5
    if kind == "infinite":
        p["W_2"] += 0.5
    else:
        p["W_2"].fill_diagonal_(0.5)
    if bf16:
        p = {n: v.bfloat16() if n[0] == "W" else v for n, v in p.items()}
    dz = torch.from_numpy((rng.standard_normal((Q, da)) / Q).astype(np.float32))
    for n, v in ends.items():
        dz[:, n] = 0.0
        dz[Q // 2, n] = v
    mem = torch.zeros(3, dm, dtype=torch.bfloat16 if bf16 else torch.float32)
    i32 = dict(dtype=torch.int32)
    _, g, _ = _forward_backward(p, mem, None, torch.zeros(Q, **i32), torch.zeros(Q), torch.full((Q, k), -1, **i32),
                                torch.zeros(Q, k), torch.zeros(Q, k, **i32), torch.zeros(dm), torch.zeros(dm), dz, H, k,
                                torch.zeros(1, **i32), bf16)
    want = dz.double().sum(0)
    for name, slope in (("W_2", 0.5), ("b_2", 1.0)) + ((("b_1", 0.5),) if kind == "largest" else ()):
        got, ref = g[name].double(), slope * want
        for n in ends:
            assert (got[n] == ref[n]).all(), (name, n, got[n], ref[n])
        rest = [n for n in range(da) if n not in ends]
        scale = slope * dz[:, rest].abs().double().sum(0)
        err = ((got.view(da, -1) - ref[:, None])[rest] / scale[:, None]).abs().max().item()
        assert err <= 1e-6, (name, err)
    if kind == "infinite":
        assert (g["b_1"] == -math.inf).all()


def _scored(scores, values, k):
    """Queries whose slot j of row i has the score scores[i, j] and the value values[i, j] in the first head's first
    column, all exact: u is one memory column's 2^100 (the score times 8 over it, head width 64; -inf: a product past
    the range), the value another.  The arguments of _forward_backward up to the time encoder."""
    Q, dm, dt, da = scores.shape[0], 4, 4, 128
    p = _passing(dm, dt, da)
    p["b_q"][0] = p["W_k"][0, 0] = 2.0 ** 50
    p["W_v"][0, 1] = 1.0
    mem = torch.zeros(Q * k, dm)
    mem[:, 0] = torch.where(scores < -1e38, -(2.0 ** 40), scores * 2.0 ** -97).reshape(-1)
    mem[:, 1] = values.reshape(-1)
    i32 = dict(dtype=torch.int32)
    return (p, mem, None, torch.zeros(Q, **i32), torch.zeros(Q), torch.arange(Q * k, **i32).view(Q, k), torch.zeros(Q, k),
            torch.zeros(Q, k, **i32), torch.zeros(dt), torch.zeros(dt))


def test_softmax_error():
    """A probability between 0.5 and e^-15 against 64 bits: the exponential's (at most 1.4 ulp, 8.3e-8), the
    denominator's and the quotient's rounding (6e-8 each), 2.1e-7 in all."""
    Q = 3000
    rng = np.random.default_rng(2)
    scores = torch.zeros(Q, 2)
    scores[:, 1] = torch.from_numpy(-rng.uniform(0, 15, Q).astype(np.float32))
    values = torch.zeros(Q, 2)
    values[:, 1] = 1.0
    z, _, _ = _forward_backward(*_scored(scores, values, 2), torch.zeros(Q, 128), 2, 2, torch.zeros(1, dtype=torch.int32))
    want = 1.0 / (1.0 + torch.exp(-scores[:, 1].double()))
    err = ((z[:, 0].double() - want) / want).abs().max().item()
    log(f"[attn] softmax: largest relative error {err:.2e}")
    assert err <= 2.1e-7


@pytest.mark.parametrize("first", [1, 4, 5, 9])
def test_scores_below_the_range(first):
    """Leading slots whose score is -inf (a product past the float range) weigh nothing beside the others."""
    k, Q = 12, 20
    rng = np.random.default_rng(first)
    scores = torch.from_numpy(rng.uniform(-2, 2, (Q, k)).astype(np.float32))
    scores[:, :first] = -math.inf
    values = torch.from_numpy(rng.uniform(-1, 1, (Q, k)).astype(np.float32))
    z, g, d_mem = _forward_backward(*_scored(scores, values, k), torch.ones(Q, 128) / Q, 2, k,
                                    torch.arange(Q * k, dtype=torch.int32))
    w = torch.softmax(scores[:, first:].double(), 1)
    err = rel_err(z[:, 0].numpy(), (w * values[:, first:].double()).sum(1).numpy())
    log(f"[attn] {first} leading scores of -inf: error {err:.1e}")
    assert err <= 1e-6
    assert all(torch.isfinite(v).all() for v in g.values()) and torch.isfinite(d_mem).all()


@pytest.mark.parametrize("H", [2, 4])   # four heads: the general path
@pytest.mark.parametrize("Q", [2_000, 60_000])
def test_weight_gradient_of_columns_that_hardly_vary(H, Q):
    """W_2's gradient where every row's a1 is the same and its dz column varies by a tenth: a long sum of nearly
    equal terms, whose roundings must not all go one way.  Error of the whole against 64 bits (2-norm): the result's
    own rounding 3.4e-8, the partial sums' that of a few float32 additions more; with roundings that do not
    average out it grows past 2e-7."""
    dm, da, k = 4, 100, 1
    log(f"[attn] nearly constant columns: H {H} queries {Q}")
    rng = np.random.default_rng(H + Q)
    p = {n: torch.zeros(*s) for n, s in dict(W_q=(da, 2 * dm), W_k=(da, 2 * dm), W_v=(da, 2 * dm), W_o=(da, da),
                                             W_1=(da, da + dm), W_2=(da, da)).items()}
    p.update({"b" + n[1:]: torch.zeros(da) for n in list(p)})
    p["b_1"] = torch.from_numpy(rng.uniform(0.5, 1.0, da).astype(np.float32))
    dz = torch.from_numpy((rng.uniform(0.5, 1.0, da) * (1 + 0.1 * rng.standard_normal((Q, da))) / Q).astype(np.float32))
    i32 = dict(dtype=torch.int32)
    _, g, _ = _forward_backward(p, torch.zeros(3, dm), None, torch.zeros(Q, **i32), torch.zeros(Q),
                                torch.full((Q, k), -1, **i32), torch.zeros(Q, k), torch.zeros(Q, k, **i32),
                                torch.zeros(dm), torch.zeros(dm), dz, H, k, torch.zeros(1, **i32))
    ref = torch.outer(dz.double().sum(0), p["b_1"].double())
    err = ((g["W_2"].double() - ref).norm() / ref.norm()).item()
    log(f"  error {err:.2e}")
    assert err <= 1.0e-7


def test_time_gradient_sums():
    """The time encoder's gradient over 60,000 slots whose sine is 1 (arguments of pi / 2): sums of terms of one sign, in
    64 bits from the blocks' partials on, so the result's own rounding (2.5e-8 on average) is what is left."""
    dm, dt, da, Q = 4, 64, 128, 60_000
    rng = np.random.default_rng(9)
    p = _passing(dm, dt, da)
    i = torch.arange(dt)
    p["W_v"][i, dm + i] = 1.0
    tb = torch.full((dt,), np.float32(np.pi / 2))
    q_t = torch.from_numpy(rng.uniform(1, 1000, Q).astype(np.float32))
    dz = torch.zeros(Q, da)
    dz[:, :dt] = torch.from_numpy((rng.uniform(0.5, 1.0, dt) * (1 + 0.3 * rng.standard_normal((Q, dt))) / Q).astype(np.float32))
    i32 = dict(dtype=torch.int32)
    _, g, _ = _forward_backward(p, torch.zeros(2, dm), None, torch.zeros(Q, **i32), q_t, torch.ones(Q, 1, **i32),
                                torch.zeros(Q, 1), torch.zeros(Q, 1, **i32), torch.zeros(dt), tb, dz, 1, 1,
                                torch.zeros(1, **i32))
    d = dz[:, :dt].double()
    for name, ref in (("time_b", -d.sum(0)), ("time_w", -(d * q_t.double()[:, None]).sum(0))):
        err = ((g[name].double() - ref) / ref).pow(2).mean().sqrt().item()
        log(f"[attn] {name} over {Q} slots: error {err:.2e}")
        assert err <= 3.5e-8, name
