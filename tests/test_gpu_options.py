"""GPU parity under non-default options: every tunable of kfac_options that changes which kernels run, how the
contractions are split or how the work is spread over streams must leave the results within the same tolerances
against the float64 oracle (fused step and separate calls)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2002_06015_amd import kfac, workloads as wl

pytestmark = pytest.mark.gpu

TOL_FACTOR = 1e-4
TOL_INVERSE = 1e-3      # the group holds a 601 x 601 factor inverted through the recursion
TOL_PRECOND = 1e-3
GAMMA = 0.05

# a recursion of two levels (601 -> 300 -> 150), the correlation form over several tiles, long contractions
# (split along K under the default rules), a strided 7 x 7 layer through patches, a tiny layer
LAYERS = [wl.fc_layer(8, 600, 300), wl.conv_layer(2, 40, 130, 3, 1, 1, 10), wl.conv_layer(4, 160, 130, 1, 1, 0, 8),
          wl.conv_layer(32, 16, 24, 1, 1, 0, 28), wl.conv_layer(2, 3, 8, 7, 2, 3, 32), wl.fc_layer(5, 7, 3, bias=0)]

OPTIONS = [
    {"force_tile": 64},
    {"force_tile": 128},
    {"recursion_leaf": 64},                                   # four levels, the smallest leaf kernel
    {"recursion_leaf": 200},                                  # the middle leaf kernel
    {"min_k_per_split": 32, "max_k_per_workgroup": 64, "target_workgroups": 4096},   # as many splits as the rules allow
    {"target_workgroups": 1, "max_k_per_workgroup": 1 << 20},                          # none
    {"group_by_depth": 0},
    {"streams": 4, "early_n": 100, "staging_slots": 2},
    {"streams": 1},
    {"correlation_form": 0, "force_tile": 64},
]


def relerr(got, ref):
    got = np.asarray(got, dtype=np.float64)
    ref = np.asarray(ref, dtype=np.float64)
    return float(np.abs(got - ref).max() / max(np.abs(ref).max(), 1e-300))


def host(t):
    return t.detach().float().cpu().numpy().astype(np.float64)


@pytest.fixture(scope="module")
def gpu():
    assert torch.cuda.is_available()
    torch.cuda.set_device(0)
    kfac.lib()
    return torch.device("cuda")


@pytest.fixture(scope="module")
def reference():
    acts = [wl.make_act(L, 900 + i) for i, L in enumerate(LAYERS)]
    grads = [wl.make_grad_out(L, 900 + i) for i, L in enumerate(LAYERS)]
    gws = [wl.make_grad_W(L, 900 + i) for i, L in enumerate(LAYERS)]
    ref = []
    for i, L in enumerate(LAYERS):
        Ar, Gr = oracle.kfac_stats(tuple(L), acts[i], grads[i], 0.0, False, None, None)
        Air, Gir, pir, info = oracle.kfac_invert(Ar, Gr, GAMMA)
        assert not info.any()
        ref.append((Ar, Gr, Air, Gir, pir, oracle.kfac_precondition(Gir, Air, gws[i])))
    return acts, grads, gws, ref


def _plain_products(ctx):
    """(variants of the products, number of reductions) of an inversion and a preconditioning of LAYERS."""
    gen = torch.Generator(device="cuda").manual_seed(1)
    spd = [[torch.eye(d, device="cuda") for d in (L.dA, L.dG)] for L in LAYERS]
    A, G = [x[0] for x in spd], [x[1] for x in spd]
    Ai, Gi = [torch.zeros_like(x) for x in A], [torch.zeros_like(x) for x in G]
    W = [torch.randn(L.dG, L.dA, device="cuda", generator=gen) for L in LAYERS]
    U = [torch.zeros_like(w) for w in W]
    pi, info = torch.zeros(len(LAYERS), device="cuda"), torch.zeros(2 * len(LAYERS), dtype=torch.int32, device="cuda")
    kfac.kfac_profile_enable(ctx, True)
    kfac.kfac_invert(ctx, LAYERS, A, G, GAMMA, Ai, Gi, pi, info)
    inv = kfac.kfac_profile_read(ctx)
    kfac.kfac_precondition(ctx, LAYERS, Gi, Ai, W, U)
    pre = kfac.kfac_profile_read(ctx)
    return [({e["variant"] for e in es if e["kernel"] == "gemm_f32_split"}, sum(e["kernel"] == "gemm_reduce" for e in es)) for es in (inv, pre)]


@pytest.mark.parametrize("fields,variants,split", [
    ({}, None, (False, False)),                                                    # nothing of this size is split by default
    ({"min_k_per_split": 32, "max_k_per_workgroup": 64, "target_workgroups": 4096}, {0, 1}, (True, True)),
    ({"target_workgroups": 1, "max_k_per_workgroup": 1 << 20}, {0, 1}, (False, False)),
    ({"force_tile": 64}, {1}, (False, False)),                                     # (contractions too short for two parts of 512)
    ({"force_tile": 64, "min_k_per_split": 128}, {1}, (True, True)),
    ({"force_tile": 128, "min_k_per_split": 128}, {0}, (True, True)),
    ({"max_k_per_workgroup": 128}, {0, 1}, (True, True)),
], ids=lambda v: ",".join("%s=%s" % kv for kv in v.items()) or "defaults" if isinstance(v, dict) else "")
def test_split_rule_holds_for_plain_products(gpu, fields, variants, split):
    """The limits of the split rule and the tile, where they are set, hold for the inversion's and the preconditioning's products."""
    ctx = kfac.Context(LAYERS, opts=kfac.options(**fields))
    for (seen, reductions), expected in zip(_plain_products(ctx), split):
        assert (reductions > 0) == expected
        assert variants is None or seen <= variants
    ctx.close()


@pytest.mark.parametrize("fields", OPTIONS, ids=lambda f: ",".join("%s=%s" % kv for kv in f.items()))
def test_results_do_not_depend_on_the_options(gpu, reference, fields):
    acts, grads, gws, ref = reference
    layers, n = LAYERS, len(LAYERS)
    d_act = [torch.from_numpy(a).cuda() for a in acts]
    d_grad = [torch.from_numpy(g).cuda() for g in grads]
    d_gw = [torch.from_numpy(g).cuda() for g in gws]
    for fused in (False, True):
        ctx = kfac.Context(layers, kfac.KFAC_F32, opts=kfac.options(**fields))
        A = [torch.full((L.dA, L.dA), float("nan"), device="cuda") for L in layers]
        G = [torch.full((L.dG, L.dG), float("nan"), device="cuda") for L in layers]
        Ai = [torch.zeros(L.dA, L.dA, device="cuda") for L in layers]
        Gi = [torch.zeros(L.dG, L.dG, device="cuda") for L in layers]
        U = [torch.zeros(L.dG, L.dA, device="cuda") for L in layers]
        pi = torch.zeros(n, device="cuda")
        info = torch.zeros(2 * n, dtype=torch.int32, device="cuda")
        if fused:
            kfac.kfac_step(ctx, layers, kfac.KFAC_F32, d_act, d_grad, 0.0, False, A, G, None, GAMMA, Ai, Gi, pi, info, d_gw, U)
        else:
            kfac.kfac_stats(ctx, layers, kfac.KFAC_F32, d_act, d_grad, 0.0, False, A, G)
            kfac.kfac_invert(ctx, layers, A, G, GAMMA, Ai, Gi, pi, info)
            kfac.kfac_precondition(ctx, layers, Gi, Ai, d_gw, U)
        torch.cuda.synchronize()
        ctx.close()
        assert not info.cpu().numpy().any()
        for i, L in enumerate(layers):
            Ar, Gr, Air, Gir, pir, Ur = ref[i]
            what = "%s layer %d %s fused=%s" % (fields, i, tuple(L), fused)
            hA, hG = host(A[i]), host(G[i])
            assert np.array_equal(hA, hA.T) and np.array_equal(hG, hG.T), what
            assert relerr(hA, Ar) <= TOL_FACTOR, what
            assert relerr(hG, Gr) <= TOL_FACTOR, what
            assert abs(float(pi[i]) - pir) <= 1e-4 * pir, what
            assert relerr(host(Ai[i]), Air) <= TOL_INVERSE, what
            assert relerr(host(Gi[i]), Gir) <= TOL_INVERSE, what
            assert relerr(host(U[i]), Ur) <= TOL_PRECOND, what
