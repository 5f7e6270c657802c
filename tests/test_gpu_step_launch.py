"""The asynchronous layer step in one launch (routing, match and experts) against the synchronous one, whose routing and match are kernels
of their own: the same picks, gate weights, matches, scores and orders, bit for bit; the output up to the order of its sums."""
import numpy as np
import pytest
import torch

from tests.helpers import EPS, dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def m():
    import paper_2401_14361_amd as mod
    mod.lib()
    return mod


def _cache(m, desc, seed):
    S = desc.L * desc.E
    cache = m.Cache(desc, S)
    cache.reset(S)
    rng = torch.Generator(device="cuda").manual_seed(seed)
    for s in range(S + desc.L * desc.n_shared):
        t = cache.slot_tensor(s)
        w = torch.randn(t.numel(), generator=rng, device="cuda") * 0.05
        t.copy_((w.to(torch.bfloat16).view(torch.int16) if desc.wdtype == m.WDTYPE_BF16 else w.view(torch.int32)).view(t.dtype))
    return cache


def _steps(m, desc, eamc, inputs, sync):
    routers, bias, x, eam0 = inputs
    cache = _cache(m, desc, 5)
    eam = eam0.clone()
    y = torch.empty((desc.L, desc.H), dtype=torch.float32, device="cuda")
    m.profile_enable(64)
    out = []
    for l in range(desc.L):
        m.moe_decode_layer(cache, eamc, eam, l, routers[l], bias[l], x[l], y[l], sync=sync)
        step = cache.last_step()
        top, sim = cache.last_matches()
        out.append(dict(step, top=top, sim1=sim, y=y[l].cpu().numpy(), eam=eam.cpu().numpy()))
    launches = len(m.profile_samples("route_topk_kernel"))
    m.profile_disable()
    assert cache.error_flags() == 0
    cache.close()
    return out, launches


# L, E, k, n_shared, H, I, wdtype, renorm, N, cell bytes, elements the router starts behind a 16-byte boundary
SHAPES = [
    (3, 300, 6, 1, 256, 40, "bf16", 0, 30, 4, 0),      # logits in LDS
    (1, 1100, 8, 0, 256, 8, "bf16", 1, 20, 4, 0),      # more than the ranking takes; more rows than wavefronts that route
    (2, 1, 1, 0, 512, 300, "bf16", 0, 5, 4, 0),        # one expert
    (3, 64, 6, 2, 2048, 352, "bf16", 0, 1000, 4, 0),   # shared experts first, all the matching workgroups
    (4, 8, 8, 0, 260, 33, "fp32", 1, 40, 4, 0),        # all experts, a row that ends inside a chunk
    (4, 160, 6, 0, 512, 24, "bf16", 0, 1, 2, 0),       # one matching workgroup: most rows in the streaming ones
    (2, 16, 2, 1, 4096, 20, "fp32", 0, 300, 4, 0),     # the longest rows: fewest wavefronts
    (2, 16, 2, 1, 5120, 300, "bf16", 1, 300, 2, 0),    # rows of ten chunks
    (3, 37, 5, 1, 768, 100, "bf16", 1, 700, 2, 1),     # single cells, router at an odd address
    (3, 8, 2, 0, 256, 64, "fp32", 1, 0, 4, 0),         # nothing to match
]


@pytest.mark.parametrize("shape", SHAPES)
def test_one_launch_is_the_synchronous_step(m, shape, monkeypatch):
    L, E, k, ns, H, I, wd, renorm, N, cell, off = shape
    bf16 = wd == "bf16"
    desc = m.ModelDesc(L, E, k, ns, H, I, m.WDTYPE_BF16 if bf16 else m.WDTYPE_FP32, renorm, EPS)
    dt = torch.bfloat16 if bf16 else torch.float32
    g = torch.Generator(device="cuda").manual_seed(L * E + H)
    flat = (torch.randn(L * E * H + off, generator=g, device="cuda") * 0.05).to(dt)
    routers = flat[off:].view(L, E, H)
    bias = torch.randn((L, E), generator=g, device="cuda")
    x = torch.randn((L, H), generator=g, device="cuda").to(dt)
    rng = np.random.default_rng(E)
    eam0 = dev(rng.integers(0, 60, (L, E)).astype(np.int32))
    eamc = m.Eamc(desc, max(N, 4), cell)
    if N:
        eamc.load(rng.integers(0, 200, (N, L, E)).astype(np.int32))
    inputs = (routers, bias, x, eam0)
    want, n = _steps(m, desc, eamc, inputs, True)
    assert n >= L
    got, n = _steps(m, desc, eamc, inputs, False)
    assert n == 0  # no launch of its own for the routing
    monkeypatch.setenv("MOEI_STEP_SPIN", "0")  # every workgroup forms the logits itself
    alone, _ = _steps(m, desc, eamc, inputs, False)
    for l in range(L):
        for key in ("eam", "w", "sim", "top", "sim1", "P", "V", "pf_order", "ev_order"):
            assert np.array_equal(got[l][key], want[l][key]), (l, key)
        # sums of at most (k + n_shared) * I products of two rounded factors, in another order
        scale = np.abs(want[l]["y"]).max()
        assert np.abs(got[l]["y"] - want[l]["y"]).max() <= 2.0 ** -24 * 4 * np.sqrt((k + ns) * I + H) * scale, l
        for key in ("eam", "w", "sim", "top", "P", "V", "pf_order", "ev_order", "y"):
            assert np.array_equal(alone[l][key], got[l][key]), (l, key)
    eamc.close()
