"""The tile shapes of the grouped SwiGLU GEMM and the always-on expert's place in its
launches, at the sizes where they can go wrong: tile edges, remainders, K loops shorter than
the copy lookahead, operands beyond 32-bit byte offsets.  Every row against the fp64
definition, with the layer's bar (bf16 rounding of activation and output)."""
from __future__ import annotations

import re

import numpy as np
import pytest

import oracle
from gpu_common import layer_tolerance_check, note, require_gpu
from synth.device import bf16_bits, state_tensors, to_device
from synth.workloads import bf16_bits_from_f32, make_fuzz_workload

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    return require_gpu()


# T (rows of h), experts, d, f, the rows of the first experts (the rest: random below `most`)
SHAPES = [
    # up to 32 tokens, 32 x 64 tiles: edges of 32 rows, partial N tiles, more rows than tokens
    (32, 40, 384, 192, [0, 1, 31, 32, 33, 65, 100], 20),
    (1, 7, 128, 64, [0, 1, 0, 1], 2),             # one token, K loops of 2 and 1 steps
    (20, 12, 256, 128, [33, 0, 32], 40),          # K loops of 4 and 2 steps
    # up to 64 tokens, 64 x 128 tiles
    (64, 24, 384, 320, [0, 1, 63, 64, 65, 129, 200], 70),
    (50, 256, 128, 64, [64, 0, 65], 10),          # 256 experts, K loops of 2 and 1 steps
    # few 256-row tiles: 32-row and 64-row tiles with many rows an expert
    (300, 3, 256, 64, [500, 0, 33], 10),
    (1200, 5, 640, 320, [512, 511, 1, 0, 257], 10),
    # 256 x 256, 128 x 256 and 64 x 128 tiles, by the pair capacity
    (900, 100, 640, 320, [0, 1, 31, 33, 255, 256, 257, 511, 512, 513, 700], 120),
    (200, 160, 128, 64, [256, 257, 0, 1], 40),    # K loops of 2 and 1 steps
    (200, 256, 256, 128, [300, 0, 255], 30),      # K loops of 4 and 2 steps
    (100, 140, 640, 320, [0, 1, 31, 32, 33, 63, 64, 65, 96, 97, 127, 128, 129, 192, 193], 50),
    # few tiles, weights past 8 MB: 128-row tiles from the pair capacity alone (400 pairs an expert)
    (500, 8, 768, 832, [400, 0, 1, 129, 257, 128], 400),
]


# capacity: the pairs + 5, or this many per expert (past 32: 128-row tiles, past 192: 256-row ones)
@pytest.mark.parametrize("per_expert", [0, 40, 200])
@pytest.mark.parametrize("case", range(len(SHAPES)))
def test_tile_shapes(torch, case, per_expert):
    from paper_2608_01784_amd import _lib as L
    T, E, d, f, first, most = SHAPES[case]
    rng = np.random.default_rng([case, 41])
    counts = rng.integers(0, most, E)
    counts[:len(first)] = first
    P = int(counts.sum())
    eo = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    st = rng.integers(0, T, P).astype(np.int32)

    def bf16(shape, scale):
        return bf16_bits_from_f32((rng.standard_normal(shape) * scale).astype(np.float32))

    h, wg, wu = bf16((T, d), 1.0), bf16((E, f, d), d ** -0.5), bf16((E, f, d), d ** -0.5)
    wd = bf16((E, d, f), 0.3 * f ** -0.5)
    cap = max(P + 5, per_expert * E)
    y = torch.full((cap, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(L.reflex_swiglu_workspace_size(cap, E, f), dtype=torch.uint8, device="cuda")
    L.reflex_grouped_swiglu(to_device(h), to_device(np.concatenate([st, np.zeros(cap - P, np.int32)])),
                            to_device(eo), to_device(wg), to_device(wu), to_device(wd), y, ws)
    torch.cuda.synchronize()
    yb = bf16_bits(y)
    got, ref = [], []
    for e in np.flatnonzero(counts):
        rows = np.arange(eo[e], eo[e + 1])
        ref.append(oracle.swiglu_expert(oracle.bf16_to_f64(h[st[rows]]), oracle.bf16_to_f64(wg[e]),
                                        oracle.bf16_to_f64(wu[e]), oracle.bf16_to_f64(wd[e])))
        got.append(oracle.bf16_to_f64(yb[rows]))
    layer_tolerance_check(np.concatenate(got), np.concatenate(ref), f"T={T} E={E} d={d} f={f} P={P}")
    assert np.isnan(oracle.bf16_to_f64(yb[P:])).all()      # rows past P untouched


# T, experts, d, f, pair capacity: pair rows of the up and the down GEMM's tiles
@pytest.mark.parametrize("T,E,d,f,cap,up,down", [
    (32, 40, 256, 128, 1280, 32, 32),               # few tokens
    (64, 64, 512, 1024, 8192, 64, 64),
    (300, 160, 512, 512, 160 * 32, 64, 64),         # few pairs an expert
    (300, 160, 512, 512, 160 * 32 + 1, 128, 128),   # up to 192, past them
    (300, 160, 512, 512, 160 * 192 + 1, 256, 256),
    (193, 8, 256, 512, 1544, 64, 32),               # few tiles: weights that stay in L2 (2 MB)
    (2048, 8, 256, 512, 8192, 64, 64),
    (193, 8, 1024, 1024, 1544, 64, 64),             # 16 MB: 64-row tiles while they run in one round
    (257, 8, 1024, 1024, 2056, 128, 64),            # up: 8 x 5 x 16 tiles on 512 places
])
def test_tile_shape_of_a_launch(torch, T, E, d, f, cap, up, down):
    # the rule that picks the tile shape, by the names of the kernels that a call launches
    from torch.profiler import ProfilerActivity, profile
    from paper_2608_01784_amd import _lib as L

    def zeros(*shape, dtype=torch.bfloat16):
        return torch.zeros(shape, dtype=dtype, device="cuda")

    args = (zeros(T, d), zeros(cap, dtype=torch.int32), zeros(E + 1, dtype=torch.int32), zeros(E, f, d),
            zeros(E, f, d), zeros(E, d, f), zeros(cap, d),
            zeros(L.reflex_swiglu_workspace_size(cap, E, f), dtype=torch.uint8))
    L.reflex_grouped_swiglu(*args)
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        L.reflex_grouped_swiglu(*args)
        torch.cuda.synchronize()
    rows = {}
    for e in prof.events():
        m = re.search(r"swiglu_gemm_kernel<(true|false), .*Shape<(\d+), (\d+),", e.name)
        if m:
            rows[m[1]] = 32 * int(m[2]) * int(m[3])
    assert rows == {"true": up, "false": down}


@pytest.mark.parametrize("which", ["up", "down"])
def test_operands_past_32_bit_offsets(torch, which):
    # 2^30 elements or more: the input rows go through 64-bit addresses.  up: tokens at the
    # far end of a 2^20 x 1024 h; down: 2^20 activation rows of width 1024.
    from paper_2608_01784_amd import _lib as L
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    T, d, f, E = (1 << 20, 1024, 64, 2) if which == "up" else (500, 128, 1024, 2)
    P = 700 if which == "up" else (1 << 20) + 300

    def normal(shape, scale):
        return (torch.randn(shape, generator=g, device="cuda") * scale).to(torch.bfloat16)

    h = torch.empty((T, d), dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    wg, wu = normal((E, f, d), d ** -0.5), normal((E, f, d), d ** -0.5)
    wd = normal((E, d, f), 0.3 * f ** -0.5)
    st = torch.randint(max(0, T - 1000), T, (P,), generator=g, device="cuda", dtype=torch.int32)
    cut = P // 2 + 17
    eo = torch.tensor([0, cut, P], dtype=torch.int32, device="cuda")
    y = torch.empty((P, d), dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(L.reflex_swiglu_workspace_size(P, E, f), dtype=torch.uint8, device="cuda")
    print(f"operands past 32-bit offsets: {which}", flush=True)
    L.reflex_grouped_swiglu(h, st, eo, wg, wu, wd, y, ws)
    torch.cuda.synchronize()
    rows = np.unique(np.concatenate([np.linspace(0, P - 1, 400).astype(np.int64),
                                     np.arange(cut - 3, cut + 3), np.arange(P - 40, P)]))
    pick = torch.from_numpy(rows).cuda()
    x = h[st[pick].long()].double().cpu().numpy()
    ref = np.empty((len(rows), d))
    for e, m in ((0, rows < cut), (1, rows >= cut)):
        ref[m] = oracle.swiglu_expert(x[m], *(w[e].double().cpu().numpy() for w in (wg, wu, wd)))
    layer_tolerance_check(y[pick].double().cpu().numpy(), ref, f"{which} past 32-bit offsets")


@pytest.mark.parametrize("T,E,kmax,fs", [
    (24, 64, 12, 128),      # rides, 32-row tiles
    (60, 256, 12, 128),     # rides, 64-row tiles
    (105, 256, 12, 128),    # rides, 64-row tiles past 64 tokens
    (107, 256, 12, 128),    # just past the rule: launches of its own, tiles cut to 128 rows
    (40, 16, 4, 192),       # another width: launches of its own, 64-row tiles
    (2100, 16, 4, 128),     # launches of its own, tiles cut to 128 rows
    (4100, 16, 4, 128),     # launches of its own, past 4096 rows, still cut
    (600, 16, 4, 5504),     # up: 129 tiles if not cut, 256-row tiles; down: one N tile, cut
    (8400, 8, 2, 192),      # past an eighth of 256 CUs: 256-row tiles (4100 rows: cut)
])
@pytest.mark.parametrize("no_pairs", [False, True])
def test_always_on_expert(torch, T, E, kmax, fs, no_pairs):
    from paper_2608_01784_amd.layer import ExpertWeights, MoELayer, TokenState
    w = make_fuzz_workload(300 + T, T=T, d=256, E=E, f=128, f_shared=fs, k_max=kmax)
    dw = {"w_gate": to_device(w.w_gate()), "w_up": to_device(w.w_up()), "w_down": to_device(w.w_down()),
          "w_router": to_device(w.w_router()),
          "router_bias": None if w.router_bias is None else to_device(w.router_bias)}
    shared = w.shared_weights()
    dw["ws_gate"], dw["ws_up"], dw["ws_down"] = (to_device(x) for x in shared)
    lay = MoELayer(w.T, w.d, ExpertWeights(**dw), w.params)
    st = TokenState(**state_tensors(w))
    k_in = np.zeros(w.T, np.int32) if no_pairs else None
    out = lay.forward(to_device(w.h), st, k_in=None if k_in is None else to_device(k_in))
    torch.cuda.synchronize()
    assert int(lay.pairs.item()) == (0 if no_pairs else int(lay.k.sum().item()))
    k = np.zeros(w.T, np.int64) if no_pairs else lay.k.cpu().numpy()
    route = oracle.topk_route(lay.logits.cpu().numpy().astype(np.float64), k)
    wg, wu, wd = w.w_gate(), w.w_up(), w.w_down()
    toks = np.arange(w.T) if T < 1000 else np.unique(np.linspace(0, w.T - 1, 600).astype(int))
    ref = oracle.moe_layer(w.h, route, lambda e: (wg[e], wu[e], wd[e]), w.E, shared=shared, tokens=toks)
    layer_tolerance_check(oracle.bf16_to_f64(bf16_bits(out))[toks], ref,
                          f"always-on expert T={T} E={E} fs={fs} no_pairs={no_pairs}")
    note("ok")


# K_max = 1 and 0 (no routed pair at all): the always-on expert's rows, not the pairs, are what
# the launch works on; riding up to five tokens per expert, launches of its own above
@pytest.mark.parametrize("kmax,T", [(1, 80), (1, 81), (0, 1), (0, 80), (0, 81), (0, 2100), (0, 4100)])
def test_always_on_expert_with_few_or_no_pairs(torch, kmax, T):
    from paper_2608_01784_amd.layer import ExpertWeights, MoELayer, TokenState
    w = make_fuzz_workload(600 + T, T=T, d=256, E=16, f=128, f_shared=128, k_max=1)
    params = w.params.replace(k_min=min(kmax, w.params.k_min), k_max=kmax)
    shared = w.shared_weights()
    lay = MoELayer(w.T, w.d, ExpertWeights(
        w_gate=to_device(w.w_gate()), w_up=to_device(w.w_up()), w_down=to_device(w.w_down()),
        w_router=to_device(w.w_router()),
        router_bias=None if w.router_bias is None else to_device(w.router_bias),
        ws_gate=to_device(shared[0]), ws_up=to_device(shared[1]), ws_down=to_device(shared[2])), params)
    out = lay.forward(to_device(w.h), TokenState(**state_tensors(w)))
    torch.cuda.synchronize()
    k = lay.k.cpu().numpy()
    assert k.max(initial=0) <= kmax and int(lay.pairs.item()) == k.sum()
    route = oracle.topk_route(lay.logits.cpu().numpy().astype(np.float64), k)
    wg, wu, wd = w.w_gate(), w.w_up(), w.w_down()
    toks = np.unique(np.linspace(0, w.T - 1, 600).astype(int))
    ref = oracle.moe_layer(w.h, route, lambda e: (wg[e], wu[e], wd[e]), w.E, shared=shared, tokens=toks)
    layer_tolerance_check(oracle.bf16_to_f64(bf16_bits(out))[toks], ref, f"K_max {kmax}, T={T}")


@pytest.mark.parametrize("big,rest", [(257, 3), (1000, 10), (129, 30), (300, 128)])
def test_few_large_experts(torch, big, rest):
    # 256-row tiles cut to 128 rows where few experts have far more rows than the others
    # (the first three; in the fourth no expert has four times the mean)
    from paper_2608_01784_amd import _lib as L
    rng = np.random.default_rng(big)
    T, E, d, f = 1100, 192, 256, 128
    counts = np.full(E, rest)
    counts[[5, 77]] = [big, max(rest, big // 2 + 1)]
    counts[100:110] = 0
    P = int(counts.sum())
    eo = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    st = rng.integers(0, T, P).astype(np.int32)

    def bf16(shape, scale):
        return bf16_bits_from_f32((rng.standard_normal(shape) * scale).astype(np.float32))

    h, wg, wu = bf16((T, d), 1.0), bf16((E, f, d), d ** -0.5), bf16((E, f, d), d ** -0.5)
    wd = bf16((E, d, f), 0.3 * f ** -0.5)
    cap = 200 * E        # (256-row tiles)
    st = np.concatenate([st, np.zeros(cap - P, np.int32)])
    y = torch.full((cap, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(L.reflex_swiglu_workspace_size(cap, E, f), dtype=torch.uint8, device="cuda")
    L.reflex_grouped_swiglu(to_device(h), to_device(st), to_device(eo), to_device(wg), to_device(wu),
                            to_device(wd), y, ws)
    torch.cuda.synchronize()
    yb = bf16_bits(y)[:P]
    ref = np.concatenate([oracle.swiglu_expert(oracle.bf16_to_f64(h[st[eo[e]:eo[e + 1]]]),
                                               *(oracle.bf16_to_f64(w[e]) for w in (wg, wu, wd)))
                          for e in np.flatnonzero(counts)])
    layer_tolerance_check(oracle.bf16_to_f64(yb), ref, f"experts of {big} and {rest} rows")


@pytest.mark.parametrize("T,E,B,d", [(2048, 64, 1, 1024), (512, 256, 300, 1024), (520, 256, 2, 1024),
                                     (16384, 256, 1000, 128), (4100, 64, 5, 512),
                                     # the small tiles' launch past 2^17 scores (an odd number of slices)
                                     (2100, 64, 3, 768), (513, 256, 300, 1280), (512, 256, 2, 512)])
def test_counts_beside_the_scores(torch, T, E, B, d):
    # the launch of large score tiles computes the counts of B sequences in its first
    # workgroups: more sequences than tiles, empty sequences, one sequence of several slices
    from paper_2608_01784_amd.layer import ExpertWeights, MoELayer, TokenState
    from gpu_common import oracle_budget
    w = make_fuzz_workload(400 + B, T=T, d=d, E=E, f=64, k_max=8)
    rng = np.random.default_rng(B)
    cuts = np.sort(rng.integers(0, T + 1, B - 1)) if B > 1 else np.zeros(0, int)
    w.seq_offsets = np.concatenate([[0], cuts, [T]]).astype(np.int32)
    w.active_block = rng.integers(1, 5, B).astype(np.int32)
    dw = {"w_gate": to_device(w.w_gate()), "w_up": to_device(w.w_up()), "w_down": to_device(w.w_down()),
          "w_router": to_device(w.w_router()),
          "router_bias": None if w.router_bias is None else to_device(w.router_bias)}
    lay = MoELayer(w.T, w.d, ExpertWeights(**dw), w.params)
    lay.forward(to_device(w.h), TokenState(**state_tensors(w)))
    torch.cuda.synchronize()
    assert np.array_equal(lay.k.cpu().numpy(), oracle_budget(w).k)
    toks = np.unique(np.linspace(0, T - 1, 500).astype(int))
    ref = oracle.bf16_to_f64(w.h[toks]) @ w.w_router().astype(np.float64).T
    if w.router_bias is not None:
        ref = ref + w.router_bias
    got = lay.logits.cpu().numpy()[toks]
    assert (np.abs(got - ref).max(1) <= 1e-4 * np.abs(ref).max(1)).all()


@pytest.mark.parametrize("T,E", [(1024, 16), (1025, 16), (16401, 1), (9000, 3), (700, 24), (2705, 96),
                                 (4096, 64), (4097, 64), (65, 256), (1024, 256), (1040, 256)])
def test_pair_sort_launches(torch, T, E):
    # the pair sort inside the route launch up to 1024 (16-token block, expert) counts, in
    # one launch up to 16384, in two above: both sides of each line, expert counts that
    # share a wave, straddle two and leave lanes empty
    from test_gpu_parity import _fused_routing, _fuzz_layer
    w = make_fuzz_workload(T, T=T, d=128, E=E, f=64, k_max=min(E, 12))
    lay, st = _fuzz_layer(torch, w)
    for k in (None, np.random.default_rng(T).integers(0, w.params.k_max + 1, T) * (np.arange(T) % 40 < 25)):
        lay.forward(to_device(w.h), st, k_in=None if k is None else to_device(k.astype(np.int32)))
        torch.cuda.synchronize()
        route = oracle.topk_route(lay.logits.cpu().numpy().astype(np.float64),
                                  lay.k.cpu().numpy() if k is None else k)
        ref = oracle.pair_permutation(route.token, route.expert, E)
        got, P = _fused_routing(torch, lay, w), int(route.offsets[-1])
        assert np.array_equal(got["pair_offsets"], route.offsets)
        assert np.array_equal(got["pair_expert"][:P], route.expert)
        assert np.array_equal(got["expert_offsets"], ref.expert_offsets)
        assert np.array_equal(got["sorted_token"][:P], ref.sorted_token)
        assert np.array_equal(got["pair_to_sorted"][:P], ref.pair_to_sorted)


# finished scores, the small score tiles' K slices (two of 256 columns) and the large tiles' (four)
@pytest.mark.parametrize("T,d", [(100, 384), (100, 512), (2048, 1024)])
@pytest.mark.parametrize("counts", ["uniform", "topp", "threshold", "budget"])
def test_forward_without_the_optional_outputs(torch, T, d, counts):
    # with no buffers for scores, counts and pair count the forward keeps them in its workspace
    # (a count rule's finished scores then lie over the first K slice's partials): the same
    # output and routing, bit for bit, as with them
    from paper_2608_01784_amd import _lib as L
    from test_gpu_parity import _fused_routing, _fuzz_layer
    w = make_fuzz_workload(700 + T, T=T, d=d, E=64, f=64, k_max=12)
    lay, st = _fuzz_layer(torch, w)
    lay.k_rule, lay.k_threshold = {"topp": (1, 0.2), "threshold": (2, 0.02)}.get(counts, (0, 0.0))
    if counts == "uniform":
        lay.uniform_k = lay.kcap = 7
    h = to_device(w.h)
    a = lay.args(h, st)
    got = []
    for drop in (False, True):
        if drop:
            a.k_out = a.pairs_out = a.logits_out = None
        lay.ws.fill_(0xff)
        lay.out.fill_(float("nan"))
        L.reflex_moe_forward(a, lay.ws)
        torch.cuda.synchronize()
        routing = _fused_routing(torch, lay, w)
        P = int(routing["pair_offsets"][-1])
        assert P == int(lay.pairs.item()) == int(lay.k.sum().item()) > 0
        got.append((bf16_bits(lay.out), {n: v if n.endswith("offsets") else v[:P] for n, v in routing.items()}))
    assert np.array_equal(got[0][0], got[1][0])
    for name in got[0][1]:
        assert np.array_equal(got[0][1][name].view(np.int32), got[1][1][name].view(np.int32)), name
