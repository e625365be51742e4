"""GPU parity of the step schedule and the block stack (Sec. 3.1 Eq. 1/2,
Sec. 3.3 step-latent scheduling): the two halves of the selection against
the whole, and stacks of cached blocks over multi-step trajectories against
the oracle (schedule decisions exact, outputs within the block tolerance
times the number of stacked blocks)."""
import numpy as np
import pytest
import torch

import synth
from oracle import select as OS
from oracle.schedule import Schedule, stack_trajectory
from paper_2608_02474_amd import api

from gpu_util import (TOL_BF16_ABS, TOL_BF16_REL_L2, TOL_F32_ABS, device, down, params_to_device, say,
                      tdtype, up)

pytestmark = pytest.mark.gpu

RAGGED = synth.Workload("ragged_bf16_300tok", T=3, grid=(10, 10), D=256, H=2, F=512,
                        n_samples=4000, ratio=0.37, dtype="bf16", audio="bursts", seed=21)


@pytest.mark.parametrize("w", [synth.SMALL, synth.WAN14B_480P], ids=lambda w: w.name)
def test_saliency_then_topk_is_select(w):
    xref, x = synth.make_latents(w)
    audio = synth.make_audio(w.audio, w.n_samples, w.sample_rate, w.seed)
    dt = tdtype(w.dtype)
    X, XR = up(x, dt), up(xref, dt)
    _, _, fw = api.energy(up(audio), w.T, w.sample_rate, w.n_fft, w.hop, w.n_bands)
    whole = api.select(X, XR, fw, w.N, k=w.K)
    a = {n: down(getattr(whole, n)).copy() for n in ("idx", "mask", "n_sel_dev", "saliency", "step_delta")}
    half = api.saliency(X, XR, fw, w.N)
    api.topk(half, w.N, w.D, dt, k=w.K)
    torch.cuda.synchronize()
    for n, v in a.items():
        got = down(getattr(half, n))
        if n == "idx":          # only the first K entries are written
            got, v = got[:w.K], v[:w.K]
        assert np.array_equal(got.view(np.uint8), v.view(np.uint8)), n


def _hard_saliency(L, kind, seed):
    """Keys that meet the edges of a digit-wise selection: specials and signed
    zeros, one value everywhere, and values that differ in the lowest bits only."""
    rng = np.random.default_rng(seed)
    if kind == "special":
        pool = np.array([np.nan, np.inf, -np.inf, 0.0, -0.0, 1e-45, -1e-45, 1.0, -1.0, 3.4028235e38], np.float32)
        s = np.where(rng.random(L) < 0.5, pool[rng.integers(0, pool.size, L)], rng.standard_normal(L))
        return s.astype(np.float32)
    if kind == "equal":
        return np.full(L, 0.25, np.float32)
    if kind == "tied":      # silent frames, then ties beside a spread in the same digit
        s = np.abs(rng.standard_normal(L)).astype(np.float32)
        s[: L // 3] = 0.0
        s[L // 3::2] = 0.7
        return s
    bits = np.float32(0.75).view(np.uint32) + rng.integers(0, 4096, L).astype(np.uint32)
    return bits.astype(np.uint32).view(np.float32)


@pytest.mark.parametrize("kind", ["special", "equal", "tied", "low_bits"])
@pytest.mark.parametrize("L", [1, 1023, 1025, 2049, 4096, 4097, 7168, 8193, 16384, 16385, 32768, 32769,
                               49152, 49153, 65536, 65537, 81920, 81921])
def test_topk_edges(L, kind):
    """Sizes at the edges of the register forms and of the shared stores (from
    5 rounds of 1024 keys) and crowded digits, against a sort by (NaN first, value, index); exact."""
    s = _hard_saliency(L, kind, L)
    order = np.lexsort((np.arange(L), -np.where(np.isnan(s), 0.0, s.astype(np.float64)), ~np.isnan(s)))
    S = up(s)
    cases = [("k", k, np.sort(order[:k])) for k in sorted({0, 1, L // 3, L - 1, L})]
    thr = float(s[~np.isnan(s)].max()) if kind == "equal" else 0.75
    cases += [("threshold", t, np.flatnonzero(np.isnan(s) | (s > np.float32(t)))) for t in (thr, -1.0)]
    for mode, v, want in cases:
        say(f"topk L={L} {kind} {mode}={v}")
        sel = api.Selection(idx=torch.full((L,), -1, dtype=torch.int32, device=device()),
                            mask=torch.full((L,), 7, dtype=torch.uint8, device=device()),
                            n_sel_dev=torch.empty(1, dtype=torch.int32, device=device()), n_sel=None,
                            saliency=S, step_delta=None)
        api.topk(sel, L, 64, torch.float32, **{mode: v})
        torch.cuda.synchronize()
        idx, mask = down(sel.idx), down(sel.mask)
        m = np.zeros(L, np.uint8)
        m[want] = 1
        assert int(sel.n_sel_dev.item()) == want.size, (mode, v)
        assert np.array_equal(idx[:want.size], want), (mode, v)
        assert (idx[want.size:] == -1).all(), (mode, v)      # nothing past the selected ones is written
        assert np.array_equal(mask, m), (mode, v)


@pytest.mark.parametrize("T,N,D", [(1, 1, 8), (3, 1, 512), (1, 5, 72), (2, 16, 64), (4, 16, 512), (1, 64, 504),
                                   (3, 21, 128), (5, 13, 64), (2, 8, 520)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_select_of_few_tokens_is_the_two_passes(T, N, D, dtype):
    """The one-launch selection of few tokens against the saliency pass and the
    digit-wise selection: the same bits, with equal rows (ties), rows without
    change, a zero reference and non-finite values."""
    L = T * N
    rng = np.random.default_rng(L * 1000 + D)
    x, xr = (rng.standard_normal((2, L, D)) * 0.7).astype(np.float32)
    for r in range(0, L, 3):
        x[r], xr[r] = x[0], xr[0]
    x[1::7] = xr[1::7]
    xr[2::11] = 0.0
    if L > 8:
        x[5, 0], x[6, D - 1], xr[8, 3] = np.nan, np.inf, np.inf
    dt = tdtype(dtype)
    X, XR, fw = up(x, dt), up(xr, dt), up(np.linspace(0.0, 1.0, T).astype(np.float32))
    half = api.saliency(X, XR, fw, N)
    thr = float(np.nanmedian(down(half.saliency)))
    for mode, v in [("k", k) for k in sorted({0, 1, L // 2, L})] + [("threshold", thr), ("threshold", -1.0)]:
        say(f"select of {L} tokens D={D} {dtype} {mode}={v}")
        whole = api.select(X, XR, fw, N, **{mode: v})
        api.topk(half, N, D, dt, **{mode: v})
        torch.cuda.synchronize()
        n = int(half.n_sel_dev.item())
        assert int(whole.n_sel_dev.item()) == n, (mode, v)
        for name in ("mask", "saliency", "step_delta", "idx"):
            a, b = down(getattr(whole, name)), down(getattr(half, name))
            if name == "idx":
                a, b = a[:n], b[:n]
            assert np.array_equal(a.view(np.uint8), b.view(np.uint8)), (mode, v, name)


def _trajectory(w, steps, seed=7):
    rng = np.random.default_rng(seed)
    from oracle.cache import cast_act
    x = rng.standard_normal((w.L, w.D)).astype(np.float32)
    out = []
    for t in range(steps):
        out.append(cast_act(x, w.dtype))
        x = (x + rng.standard_normal(x.shape) * (0.3 / (t + 1))).astype(np.float32)
    return out


def _stack_case(w, n_blocks, steps, sched: Schedule):
    blocks = [synth.make_block_weights(w.with_(seed=w.seed + 100 * b)) for b in range(n_blocks)]
    xs = _trajectory(w, steps)
    fw = np.linspace(0.3, 1.0, w.T).astype(np.float32)
    want = stack_trajectory(blocks, xs, fw, w.N, w.H, sched, w.dtype)
    dt = tdtype(w.dtype)
    stack = api.BlockStack([params_to_device(p, w.dtype) for p in blocks], w.H, w.L, w.D, device(), dt,
                           api.Scheduler(sched.n_full, sched.r_min, sched.r_max, sched.alpha,
                                         sched.refresh_delta))
    FW = up(fw)
    for t, x in enumerate(xs):
        y = stack.step(up(x, dt), FW, w.N)
        torch.cuda.synchronize()
        k, full, delta = stack.history[-1]
        wk, wfull, wdelta, wy = want[t]
        say(f"stack {w.name} x{n_blocks} step {t}: k={k} full={full} delta={delta:.6g}")
        assert (k, full) == (wk, wfull)
        if t >= sched.n_full:
            assert delta == pytest.approx(wdelta, rel=1e-12)
        got = down(y).astype(np.float64)
        err = np.abs(got - wy)
        mx, rel = float(err.max()), float(np.linalg.norm(got - wy) / np.linalg.norm(wy))
        say(f"  last block output: max|err| {mx:.3e} rel-L2 {rel:.3e}")
        if w.dtype == "f32":
            assert mx <= TOL_F32_ABS * n_blocks
        else:
            assert mx <= TOL_BF16_ABS * n_blocks and rel <= TOL_BF16_REL_L2 * n_blocks
    return stack


def test_stack_f32_schedule():
    w = synth.TINY
    st = _stack_case(w, n_blocks=3, steps=6, sched=Schedule(n_full=2, r_min=0.2, r_max=0.7, alpha=0.6))
    ks = [k for k, _, _ in st.history]
    assert ks[:2] == [w.L, w.L] and all(k < w.L for k in ks[2:])


def test_stack_f32_refresh():
    w = synth.TINY.with_(name="tiny_refresh")
    st = _stack_case(w, n_blocks=2, steps=7,
                     sched=Schedule(n_full=1, r_min=0.25, r_max=0.25, alpha=0.0, refresh_delta=0.15))
    assert any(full for _, full, _ in st.history[1:]), "the Eq. 2 refresh never fired"


def test_stack_bf16():
    _stack_case(RAGGED, n_blocks=3, steps=5, sched=Schedule(n_full=1, r_min=0.2, r_max=0.6, alpha=0.5))
