"""GPU parity of the adaptive reference cache (Sec. 3.4) against the oracle:
multi-step write sequences, compared after every step — fused outputs,
entry kinds, residual codes and scales, the reference value behind every
entry, the saliency reference xref and the number of live references."""
import numpy as np
import pytest
import torch

from oracle.cache import cast_act
from oracle.refcache import NONE, REFERENCE, RESIDUAL, RefCache, step_update
from paper_2608_02474_amd import api

from gpu_util import device, down, say, tdtype, up

pytestmark = pytest.mark.gpu

# similarities this close to tau may be decided differently by two fp64
# summation orders; the seeded cases below keep every similarity farther away
MARGIN = 1e-9


def _rows_around(rng, base, idx, chain_len, noise):
    """Rows near their chain's base row, with a per-row noise level: cosine
    similarities against a chain reference spread over (0, 1)."""
    sig = noise[idx]
    return (base[idx // chain_len] + rng.standard_normal((len(idx), base.shape[1])) * sig[:, None]
            ).astype(np.float32)


def _run(L, D, chain_len, tau, dtype, steps, seed, ratio=0.4):
    rng = np.random.default_rng(seed)
    n_chains = L // chain_len
    base = rng.standard_normal((n_chains, D)).astype(np.float32)
    noise = rng.uniform(0.2, 1.6, L).astype(np.float32)
    dt = tdtype(dtype)
    ora = RefCache(L, D, chain_len, tau, dtype)
    gpu = api.RefCache(L, D, chain_len, tau, dt, device())
    xref_o = np.zeros((L, D), np.float32)
    xref_g = torch.zeros((L, D), dtype=dt, device=device())
    for step in range(steps):
        k = L if step == 0 else max(1, int(ratio * L))
        idx = np.arange(L) if step == 0 else np.sort(rng.choice(L, k, replace=False))
        y_sel = _rows_around(rng, base, idx, chain_len, noise * (1.0 + 0.3 * step))
        x = cast_act(rng.standard_normal((L, D)).astype(np.float32), dtype)
        say(f"refcache L={L} D={D} chain={chain_len} tau={tau} {dtype} step {step} k={k}")
        y_o, xref_o = step_update(ora, x, idx, y_sel, xref_o)
        mask = np.zeros(L, np.uint8)
        mask[idx] = 1
        y_g = gpu.update(up(x, dt), up(idx.astype(np.int32)), up(mask), k, up(y_sel), xref_g)
        torch.cuda.synchronize()
        sims = np.array([ora.sims[int(l)] for l in idx])
        close = np.abs(sims - ora.tau) < MARGIN
        assert not close.any(), "a similarity lies within the fp64 margin of tau: pick another seed"
        kind_g = down(gpu.ent_kind).astype(np.int8)
        assert np.array_equal(kind_g, ora.kind), "entry kinds differ"
        res = ora.kind == RESIDUAL
        assert np.array_equal(down(gpu.codes)[res], ora.codes[res])
        assert np.array_equal(down(gpu.scale)[res].view(np.uint32), ora.scale[res].view(np.uint32))
        # the reference row behind every entry, by value (slot numbers may differ)
        pool = down(gpu.pool).astype(np.float32)
        slot = down(gpu.ent_slot)
        for l in np.flatnonzero(ora.kind != NONE):
            assert np.array_equal(pool[slot[l]], ora.refs[int(ora.ref_of[l])]), ("reference", l)
        assert gpu.live_refs() == ora.live_refs()
        assert np.array_equal(down(y_g).astype(np.float32).view(np.uint32), y_o.view(np.uint32))
        assert np.array_equal(down(xref_g).astype(np.float32), xref_o)
        say(f"  ok: {int((ora.kind == REFERENCE).sum())} references, {int(res.sum())} residuals, "
            f"{ora.live_refs()} live")
    return ora


def test_refcache_small_f32():
    _run(L=120, D=64, chain_len=10, tau=0.3, dtype="f32", steps=5, seed=1)


def test_refcache_bf16_one_frame():
    _run(L=1560, D=1536, chain_len=52, tau=0.5, dtype="bf16", steps=4, seed=2)


def test_refcache_bf16_ragged_width():
    # D not a multiple of the 1024 elements one pass of the workgroup covers
    _run(L=96, D=1160, chain_len=12, tau=0.4, dtype="bf16", steps=3, seed=3)


def test_refcache_tau_extremes():
    ora = _run(L=64, D=256, chain_len=16, tau=-2.0, dtype="bf16", steps=2, seed=4)
    assert ora.live_refs() == 64 // 16
    ora = _run(L=64, D=256, chain_len=16, tau=1.5, dtype="f32", steps=2, seed=5)
    assert (ora.kind == REFERENCE).all()


def test_refcache_full_size():
    # the 32760-token 14B-shaped block, chains of one latent-grid row (52 tokens)
    _run(L=32760, D=5120, chain_len=52, tau=0.5, dtype="bf16", steps=2, seed=6)


@pytest.mark.parametrize("D,dtype", [(256, "bf16"), (296, "bf16"), (512, "f32"), (520, "bf16"), (1016, "bf16"), (1024, "f32"), (3080, "bf16"), (5120, "f32"), (8184, "bf16"), (16384, "bf16")])
def test_refcache_row_widths(D, dtype):
    # a full row or a part of one in every register width of the update kernel
    _run(L=48, D=D, chain_len=6, tau=0.4, dtype=dtype, steps=3, seed=7)


@pytest.mark.parametrize("D", [256, 512, 768, 1024, 2048, 4096, 5120, 8192, 16384])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_refcache_register_widths(D, dtype):
    """Every register width of the update kernel, filled and one chunk of 8 short
    of it, in both types."""
    for d in (D, D - 8):
        _run(L=36, D=d, chain_len=6, tau=0.4, dtype=dtype, steps=2, seed=10)


@pytest.mark.parametrize("D,L,chain_len,dtype", [(512, 33000, 60, "f32"), (768, 43740, 54, "bf16"),
                                                 (1016, 16600, 50, "f32"), (1024, 32800, 40, "bf16"),
                                                 (2040, 16500, 60, "bf16"), (2048, 8240, 40, "f32")])
def test_refcache_rows_past_the_caches(D, L, chain_len, dtype):
    """Narrow rows of more than 64 MB, whose fresh outputs the chains write
    (fewer go through waves of their own, as in the tests above)."""
    assert L * D * (2 if dtype == "bf16" else 4) > 1 << 26
    _run(L=L, D=D, chain_len=chain_len, tau=0.5, dtype=dtype, steps=2, seed=11)


def test_refcache_nothing_rewritten():
    # no chains to scan: every row rebuilt from its entry, state untouched
    L, D = 40, 520
    rng = np.random.default_rng(8)
    gpu = api.RefCache(L, D, 8, 0.4, torch.bfloat16, device())
    xref = torch.zeros((L, D), dtype=torch.bfloat16, device=device())
    x, idx = up(rng.standard_normal((L, D)).astype(np.float32), torch.bfloat16), up(np.arange(L, dtype=np.int32))
    ones = torch.ones(L, dtype=torch.uint8, device=device())
    y0 = _rows_around(rng, rng.standard_normal((L // 8, D)), np.arange(L), 8, np.full(L, 0.8))
    gpu.update(x, idx, ones, L, up(y0), xref)
    read = gpu.update(x, idx, torch.zeros_like(ones), 0, None, xref).clone()
    ora = RefCache(L, D, 8, 0.4, "bf16")
    _, xr = step_update(ora, down(x), np.arange(L), y0, np.zeros((L, D), np.float32))
    want, _ = step_update(ora, down(x), np.zeros(0, np.int64), np.zeros((0, D), np.float32), xr)
    assert np.array_equal(down(read), want) and np.array_equal(down(xref), xr)
    assert gpu.live_refs() == ora.live_refs()
