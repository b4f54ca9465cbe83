"""Parity of moe_forward (HIP) against the CPU oracle, through the C ABI, in stages:
  (i)   gate logits within tolerance of the fp64 oracle;
  (ii)  the oracle's top-k and grouping applied to the GPU's own fp32 logits must reproduce
        topk_idx, counts, offsets, perm and inv bit for bit (float summation order cannot
        flip a routing decision that is taken on identical fp32 values);
  (iii) the oracle's expert + combine stage on that routing gives `out` within 2e-2;
  (iv)  end to end from raw inputs, excluding tokens whose k-th and (k+1)-th logits are closer
        than the logit tolerance.
"""
import numpy as np
import pytest

from workloads import moe

pytestmark = pytest.mark.gpu

LOGIT_TOL = 1e-4     # max |got - ref| / max |ref|: bf16 products are exact in fp32, K <= 1024 additions
OUT_TOL = 2e-2


@pytest.fixture(scope="module")
def dyn():
    import torch
    assert torch.cuda.is_available()
    import paper_1707_02402_amd as d
    return d


@pytest.fixture(scope="module")
def util():
    from tests import gpu_util
    return gpu_util


def kernels(*shape):
    from paper_1707_02402_amd.binding import dynb_moe_kernels
    return dynb_moe_kernels(*shape)


def stack(m):
    W1 = np.stack([m.expert_weights(e)[0] for e in range(m.E)])
    W2 = np.stack([m.expert_weights(e)[1] for e in range(m.E)])
    return W1, W2


def oracle_experts(oracle, m, r, W1, W2):
    """Expert + combine stage of the oracle on a given routing (token by token above its 64-use buffer)."""
    if m.k <= 64:
        return oracle.moe_experts(m.x, r.topk_idx, r.topk_w, W1, W2)
    return np.stack([oracle.moe_token(m.x[t], r.topk_w[t], [W1[e] for e in r.topk_idx[t]], [W2[e] for e in r.topk_idx[t]])
                     for t in range(m.T)])


def check_routing(oracle, m, aux):
    r = oracle.moe_route(aux["logits"], m.k)
    for name in ("topk_idx", "counts", "offsets", "perm", "inv"):
        got = aux[name]
        assert got.dtype == np.int32 and (got == getattr(r, name)).all(), name
    assert np.abs(aux["topk_w"] - r.topk_w).max() < 1e-5
    return r


@pytest.mark.parametrize("T,d,h,E,k,empty", [(300, 64, 96, 20, 3, 0.2), (257, 32, 32, 5, 5, 0.0), (1000, 128, 160, 70, 1, 0.1),
                                              (64, 96, 64, 300, 8, 0.5), (1, 32, 32, 2, 2, 0.0),
                                              (24, 32, 32, 2100, 3, 0.0),
                                              (40, 32, 32, 1500, 6, 0.0),      # 32 register-held logits per lane, 16-byte loads
                                              (33, 32, 32, 1027, 4, 0.0),      # the same with rows that are not 16-byte aligned
                                              (200, 64, 96, 64, 16, 0.0),      # k beyond the register-held uses
                                              (50, 32, 32, 12, 12, 0.0),       # k = E > 8: full softmax
                                              (90, 40, 72, 12, 3, 0.0),        # d, h multiples of 8 only
                                              (70, 64, 64, 200, 70, 0.0)])     # k > 64: several selections per lane
def test_small_layers_every_element(dyn, util, oracle, T, d, h, E, k, empty):
    m = moe.small(seed=T + E, T=T, d=d, h=h, E=E, k=k, empty_frac=empty)
    W1, W2 = stack(m)
    out, aux = util.moe_run(dyn, m, W1, W2)
    ref_logits = oracle.moe_logits(m.x, m.Wg, m.Wn, m.noise)
    assert util.normwise(aux["logits"], ref_logits) < LOGIT_TOL                      # (i)
    r = check_routing(oracle, m, aux)                                                # (ii)
    assert (r.counts[m.empty] == 0).all()
    ref = oracle_experts(oracle, m, r, W1, W2)                                        # (iii)
    assert util.normwise(out, ref) < OUT_TOL
    if k > 64:
        return
    # (iv) end to end: tokens with a clear margin between the k-th and (k+1)-th logit must route identically
    e2e = oracle.moe_forward(m.x, m.Wg, m.Wn, m.noise, W1, W2, k)
    if k < E:
        srt = np.sort(ref_logits, axis=1)[:, ::-1]
        clear = (srt[:, k - 1] - srt[:, k]) > 4 * LOGIT_TOL * np.abs(ref_logits).max()
    else:
        clear = np.ones(T, bool)
    assert clear.mean() > 0.5
    assert (np.sort(e2e.topk_idx[clear], 1) == np.sort(r.topk_idx[clear], 1)).all()
    assert util.normwise(out[clear], e2e.out[clear]) < OUT_TOL


@pytest.mark.parametrize("T,d,h,E,k", [(300, 64, 96, 20, 3), (1000, 128, 160, 70, 1), (200, 64, 96, 64, 16), (577, 64, 96, 3, 2)])
def test_permute_inside_the_operand_load_equals_the_separate_kernel(dyn, util, T, d, h, E, k):
    """Default: the first expert layer gathers token rows through the grouping; MOE_SEPARATE_PERMUTE writes the
    permuted copy with k_permute first.  Same arithmetic on the same rows: identical bits."""
    m = moe.small(seed=T + E, T=T, d=d, h=h, E=E, k=k, empty_frac=0.1 if E > 10 else 0.0)
    W1, W2 = stack(m)
    dev = util.moe_inputs_dev(m, W1, W2)
    args = (dev["x"], dev["Wg"], dev["Wn"], dev["noise"], dev["W1"], dev["W2"], m.k)
    a = dyn.moe_forward(*args)
    b = dyn.moe_forward(*args, flags=dyn.MOE_SEPARATE_PERMUTE)
    assert (util.to_host(a) == util.to_host(b)).all()
    with pytest.raises(dyn.DynbError) as e:
        dyn.moe_forward(*args, flags=2)
    assert e.value.name == "DYNB_E_UNSUPPORTED"


@pytest.mark.parametrize("T,E,k", [(500, 10, 1), (2000, 30, 1), (400, 16, 2)])
def test_the_separate_permute_gives_the_same_bits_where_experts_have_few_tiles_of_many_rows(dyn, util, T, E, k):
    """Wide layers whose experts hold 33 to 64 rows or more, in few tiles: sums of 512 and 1024 products, so that another order of
    summation shows in the bfloat16 results."""
    m = moe.small(seed=T + E, T=T, d=512, h=1024, E=E, k=k, zipf_s=0.2)
    W1, W2 = stack(m)
    dev = util.moe_inputs_dev(m, W1, W2)
    args = (dev["x"], dev["Wg"], dev["Wn"], dev["noise"], dev["W1"], dev["W2"], m.k)
    a, aux = dyn.moe_forward(*args, want_aux=True)
    assert ((aux.counts > 32) & (aux.counts % 64 > 32)).any()
    b = dyn.moe_forward(*args, flags=dyn.MOE_SEPARATE_PERMUTE)
    assert (util.to_host(a) == util.to_host(b)).all()


def test_noiseless_gate_and_ties(dyn, util, oracle):
    """noise = NULL drops the softplus term; duplicated gate columns give exactly equal logits: lower id wins."""
    m = moe.small(seed=9, T=128, d=64, h=64, E=16, k=4)
    m.Wg[:, 8:] = m.Wg[:, :8]                    # expert e and e+8 tie on every token
    W1, W2 = stack(m)
    out, aux = util.moe_run(dyn, m, W1, W2, noise=False)
    ref_logits = oracle.moe_logits(m.x, m.Wg, None, None)
    assert util.normwise(aux["logits"], ref_logits) < LOGIT_TOL
    assert (aux["logits"][:, 8:] == aux["logits"][:, :8]).all()
    r = check_routing(oracle, m, aux)
    assert (r.topk_idx[:, 0] < 8).all() and (r.topk_idx[:, 1] == r.topk_idx[:, 0] + 8).all()
    assert util.normwise(out, oracle.moe_experts(m.x, r.topk_idx, r.topk_w, W1, W2)) < OUT_TOL


@pytest.mark.parametrize("T,d,h,E,k", [(256, 256, 32, 128, 2),      # one tile
                                        (512, 320, 32, 256, 4),      # 2 x 2 tiles, an odd number of K-chunks
                                        (768, 1024, 32, 384, 8),     # 3 x 3 tiles
                                        (2304, 256, 32, 128, 1),     # 9 token tiles
                                        (700, 256, 32, 128, 2)])     # two whole token tiles and 188 tokens
@pytest.mark.parametrize("noisy", [True, False])
def test_wide_gate_tiles(dyn, util, oracle, T, d, h, E, k, noisy):
    """Whole 256-token x 128-expert tiles, so few of them that the 16 x 16 gate kernel takes them (more: below): every logit against the
    oracle, with and without the noise term, routing on the GPU's logits; duplicated gate columns tie exactly and the lower id wins."""
    m = moe.small(seed=T + E + d, T=T, d=d, h=h, E=E, k=k)
    if not noisy:
        m.Wg[:, 64:128] = m.Wg[:, :64]           # expert e and e+64: same tile, the other expert half of a workgroup
        m.x[3, :] = 0                            # a token whose logits all tie: experts 0 .. k-1, in that order
    W1, W2 = stack(m)
    out, aux = util.moe_run(dyn, m, W1, W2, noise=noisy)
    ref_logits = oracle.moe_logits(m.x, m.Wg, m.Wn if noisy else None, m.noise if noisy else None)
    assert util.normwise(aux["logits"], ref_logits) < LOGIT_TOL
    assert np.abs(aux["logits"] - ref_logits).max() < 4 * LOGIT_TOL * np.abs(ref_logits).max()
    if not noisy:
        assert (aux["logits"][:, 64:128] == aux["logits"][:, :64]).all()
        assert (aux["logits"][3] == 0).all() and (aux["topk_idx"][3] == np.arange(k)).all()
    r = check_routing(oracle, m, aux)
    assert util.normwise(out, oracle_experts(oracle, m, r, W1, W2)) < OUT_TOL


@pytest.mark.parametrize("T,d,h,E,k", [(3333, 256, 32, 1536, 2),     # 13 x 12 tiles and 5 tokens more, the shortest K loop
                                        (1801, 320, 32, 3072, 2),     # 7 x 24 tiles and 9 tokens, an odd number of K-chunks
                                        (2048, 1024, 8, 2048, 1),     # 8 x 16 tiles, as few as the wide kernel gets at this width with noise
                                        (1024, 1024, 8, 2048, 1),     # 4 x 16 tiles, as few without
                                        (2304, 1024, 8, 896, 1)])     # 9 x 7 tiles, one less: the 64 x 64 kernel (4 x 16 with noise, too)
@pytest.mark.parametrize("noisy", [True, False])
def test_many_wide_gate_tiles(dyn, util, oracle, T, d, h, E, k, noisy):
    """As many tiles as the wide gate kernel is chosen for; the tokens behind the last whole tile go to the 64 x 64 one."""
    test_wide_gate_tiles(dyn, util, oracle, T, d, h, E, k, noisy)


@pytest.mark.parametrize("T,d,E,noisy", [(397, 64, 801, True), (513, 128, 640, True), (641, 192, 511, False), (700, 256, 463, True), (1217, 320, 258, False),
                                         (2049, 64, 1000, False), (2049, 64, 1000, True)])
def test_gate_tiles_of_whole_chunks(dyn, util, oracle, T, d, E, noisy):
    """One to five chunks of 64 channels, tokens and experts that end inside a tile; as many tiles as two workgroups a CU hold, and more."""
    assert ("gate_stream" in kernels(T, d, 64, E, 2, noisy)) == (not noisy or (T + 63) // 64 * ((E + 63) // 64) <= 512)
    m = moe.small(seed=T + E, T=T, d=d, h=64, E=E, k=2)
    W1, W2 = stack(m)
    dev = util.moe_inputs_dev(m, W1, W2)
    _, aux = dyn.moe_forward(dev["x"], dev["Wg"], dev["Wn"] if noisy else None, dev["noise"] if noisy else None, dev["W1"], dev["W2"], 2, want_aux=True)
    x, Wg, Wn = (dev[n].double() for n in ("x", "Wg", "Wn"))
    want = x @ Wg.T
    if noisy:
        want += dev["noise"].double() * (x @ Wn.T).logaddexp(x.new_zeros(1))
    got = aux.logits if hasattr(aux, "logits") else aux["logits"]
    import torch
    got = torch.as_tensor(got).to(want.device).double()
    assert float((got - want).abs().max() / want.abs().max()) < 1e-4


@pytest.mark.parametrize("T,d,h,E,k,zipf", [(1536, 256, 512, 6, 2, 1.5),      # most groups beyond 256 rows, ragged rests
                                             (2048, 128, 256, 3, 1, 0.0),      # near-equal groups, short K loops
                                             (700, 256, 256, 2, 2, 0.0)])      # every token to both experts: 700 rows each
def test_crowded_experts(dyn, util, oracle, T, d, h, E, k, zipf):
    """Few experts with hundreds of rows each (groups of several full 64-row tiles that share weight tiles, and a
    ragged last tile): every output row against the oracle."""
    m = moe.small(seed=T + E + d, T=T, d=d, h=h, E=E, k=k, zipf_s=zipf)
    W1, W2 = stack(m)
    out, aux = util.moe_run(dyn, m, W1, W2)
    r = check_routing(oracle, m, aux)
    assert (r.counts >= 256).any() and (r.counts % 64 != 0).any()
    assert util.normwise(out, oracle_experts(oracle, m, r, W1, W2)) < OUT_TOL


EDGES = (1, 31, 32, 33, 64, 65, 96, 97, 128, 129, 160, 191, 192, 255, 256, 257, 288, 384, 385, 512, 641, 0)


@pytest.mark.parametrize("d,h,k,counts", [(256, 320, 1, EDGES + (40000, 30000)),              # 4 and 5 chunks a tile, features cut at 64
                                          (1024, 1088, 1, EDGES + (5000,)),                   # ... and behind four whole tiles of them
                                          (448, 256, 2, EDGES + (40000, 30000)),              # more than 65536 uses
                                          (512, 1024, 3, EDGES + (9000,)),
                                          (576, 1856, 1, (9000,)), (320, 256, 8, (1100,) * 8),
                                          (1024, 2048, 1, (1, 64, 128, 129, 257, 385, 0, 100) * 8),    # 2^28 bytes of weights: lone tiles past the caches
                                          (1024, 2048, 1, (1, 64, 128, 257, 100, 0, 129, 90, 40, 120) * 48)])  # 12 rounds of rests: four CUs of a die take whole tiles only
def test_crowded_experts_have_the_bits_of_the_small_tiles(dyn, util, d, h, k, counts):
    """The kernel of the crowded experts against the one with tiles of 64 rows, which MOE_SEPARATE_PERMUTE always takes: both add up the channels in
    the same order.  Experts at the edges of its kinds of tiles (32, 64, 128, 256 rows), of one row and of none; tokens whose other uses go to the
    experts behind."""
    assert "stream" in kernels(sum(counts), d, h, len(counts), k)
    bits_of_both_ways(dyn, util, d, h, k, counts)


def bits_of_both_ways(dyn, util, d, h, k, counts):
    import torch
    E = len(counts)
    g = torch.Generator(device="cuda").manual_seed(d + h)
    rnd = lambda *shape, std=1.0: (torch.randn(shape, generator=g, device="cuda") * std).to(torch.bfloat16)
    first = torch.repeat_interleave(torch.arange(E, device="cuda"), torch.tensor(counts, device="cuda"))
    first = first[torch.randperm(len(first), generator=g, device="cuda")]
    T = len(first)
    x, Wg = rnd(T, d), torch.zeros(E, d, device="cuda", dtype=torch.bfloat16)
    x[:, :E] = 0
    want = torch.zeros(E, dtype=torch.int64, device="cuda")
    for j in range(k):                                                                        # logits: 8 k for the first expert, 8 less for every next
        e = (first + j) % E
        x[torch.arange(T, device="cuda"), e] = 8.0 * (k - j)
        want += torch.bincount(e, minlength=E)
    Wg[torch.arange(E), torch.arange(E)] = 1.0
    args = (x, Wg, None, None, rnd(E, h, d, std=d ** -0.5), rnd(E, d, h, std=h ** -0.5), k)
    a, aux = dyn.moe_forward(*args, want_aux=True)
    assert (torch.as_tensor(aux.counts).cpu() == want.cpu()).all()
    b = dyn.moe_forward(*args, flags=dyn.MOE_SEPARATE_PERMUTE)
    assert torch.isfinite(a.float()).all() and a.float().abs().mean() > 0.1
    assert (util.to_host(a) == util.to_host(b)).all()


def test_a_workgroup_of_more_tiles_than_its_list_holds(dyn, util):
    """k_grouped_stream looks up 512 of a workgroup's tiles at once.  4096 experts with a rest each and 8128 features are 131072 rests' tiles, 585 or 586 for each of the 224
    workgroups that take them."""
    import torch
    E, d, h, c = 4096, 256, 8128, 64
    T = E * c + 256                                                                            # expert 77: 256 rows and 64
    assert "stream" in kernels(T, d, h, E, 1)
    g = torch.Generator(device="cuda").manual_seed(5)
    e = torch.cat([torch.arange(E, device="cuda").repeat_interleave(c), torch.full((256,), 77, device="cuda")])[torch.randperm(T, generator=g, device="cuda")]
    x = torch.randn(T, d, generator=g, device="cuda").to(torch.bfloat16)
    x[:, :128] = 0
    Wg = torch.zeros(E, d, device="cuda", dtype=torch.bfloat16)                                # an expert's logit: 8 for each of its number's two halves
    for rows, number, value in ((x, e, 8.0), (Wg, torch.arange(E, device="cuda"), 1.0)):
        at = torch.arange(len(rows), device="cuda")
        rows[at, number // 64] = value
        rows[at, 64 + number % 64] = value
    def weights(rows, cols):
        w = torch.empty(E, rows, cols, dtype=torch.bfloat16, device="cuda")
        for i in range(0, E, 256):
            w[i:i + 256] = torch.randn(256, rows, cols, generator=g, device="cuda") * cols ** -0.5
        return w
    args = (x, Wg, None, None, weights(h, d), weights(d, h), 1)
    a, aux = dyn.moe_forward(*args, want_aux=True)
    want = torch.full((E,), c, device="cuda")
    want[77] += 256
    assert (aux.counts == want).all()
    b = dyn.moe_forward(*args, flags=dyn.MOE_SEPARATE_PERMUTE)
    assert torch.isfinite(a.float()).all() and a.float().abs().mean() > 0.1
    assert (util.to_host(a) == util.to_host(b)).all()


def test_a_small_layer_does_not_wait_for_a_large_one(dyn):
    """37 tokens on one stream while another runs layers whose weights are read for 0.8 ms a launch: k_grouped_stream leaves CUs to others.  A wait for one such
    launch's end is half of a large layer's time and more, in the median; 0.07 of it where there is none."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(3)
    def layer(T, d, h, E, k):
        rnd = lambda *shape: torch.randn(shape, generator=g, device="cuda")
        w = [torch.empty(E, r, c, dtype=torch.bfloat16, device="cuda") for r, c in ((h, d), (d, h))]
        for t in w:
            for i in range(0, E, 128):
                t[i:i + 128] = rnd(*t[i:i + 128].shape) * t.shape[2] ** -0.5
        x, Wg = rnd(T, d).to(torch.bfloat16), (rnd(E, d) * d ** -0.5).to(torch.bfloat16)
        ws, out = torch.empty(dyn.moe_workspace_bytes(T, d, h, E, k), dtype=torch.uint8, device="cuda"), torch.empty_like(x)
        return lambda: dyn.moe_forward(x, Wg, None, None, *w, k, out=out, workspace=ws)
    large, small = layer(16384, 1024, 2048, 1024, 4), layer(37, 512, 1024, 256, 2)
    assert "stream" in kernels(16384, 1024, 2048, 1024, 4)
    for run in (large, small, large, small):
        run()
    torch.cuda.synchronize()
    one, other = torch.cuda.Stream(), torch.cuda.Stream()
    event = lambda: torch.cuda.Event(enable_timing=True)
    begin, end, calls = event(), event(), []
    with torch.cuda.stream(one):
        begin.record()
        for _ in range(60):
            large()
        end.record()
    while not end.query():
        with torch.cuda.stream(other):
            calls.append((event(), event()))
            calls[-1][0].record()
            small()
            calls[-1][1].record()
        other.synchronize()
    torch.cuda.synchronize()
    waits = sorted(a.elapsed_time(b) for a, b in calls[:-1])
    assert len(waits) > 20
    assert waits[len(waits) // 2] < 0.25 * begin.elapsed_time(end) / 60, (waits[len(waits) // 2], waits[-1], begin.elapsed_time(end) / 60)


@pytest.mark.parametrize("d,h,k,counts", [(64, 128, 1, (1, 2, 31, 32, 33, 0, 63, 64, 65, 127, 128, 129)),   # one chunk and two
                                          (128, 192, 2, (1, 0, 31, 33, 64, 65, 200)),             # features cut at 64
                                          (192, 1024, 1, (1, 31, 32, 33, 64, 65, 0, 130) * 12),   # three chunks in two places, sixteen in three
                                          (320, 2496, 3, (70, 0, 3)),                             # 39 chunks; 64 features of a tile's 128
                                          (512, 64, 8, (5, 60, 0, 64) * 16),
                                          (960, 704, 1, (1, 64, 0, 65) * 120),                    # more than a round of the workgroups
                                          (64, 64, 2, (1000,) * 32)])
def test_layers_of_whole_chunks_have_the_bits_of_the_general_kernel(dyn, util, d, h, k, counts):
    """k_grouped_few with two and three chunks in LDS against the kernel that MOE_SEPARATE_PERMUTE takes: both add up the channels in the same order.  Row
    tiles of 1 to 64 rows around the halves that a wave multiplies, experts without uses, one chunk to 39."""
    assert kernels(sum(counts), d, h, len(counts), k) >= {"few1", "few2"}
    bits_of_both_ways(dyn, util, d, h, k, counts)


@pytest.mark.parametrize("T,d,h,E,k,noisy,taken", [(300, 64, 128, 9, 2, True, {"few1", "few2"}), (2600, 512, 448, 6, 4, True, {"few1", "few2"}), (5000, 576, 1024, 4, 4, True, {"stream"}),
                                                   (700, 256, 64, 463, 2, True, {"gate_stream"}), (650, 128, 64, 500, 1, False, {"gate_stream"})])
def test_inputs_between_16_byte_borders(dyn, util, T, d, h, E, k, noisy, taken):
    """Tensors that start 4 bytes behind a border of 16 take the kernels that load registers: the logits and results of aligned copies, bit for bit."""
    import torch
    assert taken <= kernels(T, d, h, E, k, noisy)
    g = torch.Generator(device="cuda").manual_seed(T)
    def rnd(*shape, std=1.0):
        n = int(np.prod(shape))
        return (torch.randn(n + 8, generator=g, device="cuda") * std).to(torch.bfloat16)[2:n + 2].view(shape)
    args = [rnd(T, d), rnd(E, d), rnd(E, d, std=0.1), torch.randn(T, E, generator=g, device="cuda") if noisy else None, rnd(E, h, d, std=d ** -0.5), rnd(E, d, h, std=h ** -0.5)]
    assert all(t.data_ptr() % 16 == 4 for t in args if t is not None and t.dtype == torch.bfloat16)
    aligned = [t if t is None else t.clone() for t in args]
    def both(*tensors):
        out, aux = dyn.moe_forward(*tensors, k, want_aux=True)
        return util.to_host(out), util.to_host(aux.logits)
    want = both(*aligned)
    assert all((a == b).all() for a, b in zip(both(*args), want))
    for i in (0, 1, 2, 4, 5):
        assert all((a == b).all() for a, b in zip(both(*[args[j] if j == i else aligned[j] for j in range(6)]), want)), i


def full_layer(dyn, util, m):
    """Runs a benchmark-size layer with per-expert generated weights; returns (out, aux, device inputs)."""
    import torch
    W1b = np.empty((m.E, m.h, m.d), np.uint16)
    W2b = np.empty((m.E, m.d, m.h), np.uint16)
    m.all_expert_weights_bits(W1b, W2b, threads=16)
    dev = util.moe_inputs_dev(m, np.zeros((1, 1, 1), np.float32), np.zeros((1, 1, 1), np.float32))
    dev["W1"] = torch.from_numpy(W1b.view(np.int16)).cuda().view(torch.bfloat16)
    dev["W2"] = torch.from_numpy(W2b.view(np.int16)).cuda().view(torch.bfloat16)
    out, aux = util.moe_run(dyn, m, dev=dev)
    out2, aux2 = util.moe_run(dyn, m, dev=dev)
    assert (out2 == out).all() and (aux2["perm"] == aux["perm"]).all()               # deterministic
    sep = dyn.moe_forward(dev["x"], dev["Wg"], dev["Wn"], dev["noise"], dev["W1"], dev["W2"], m.k,
                          flags=dyn.MOE_SEPARATE_PERMUTE)
    assert (util.to_host(sep) == out).all()              # permute as its own kernel or inside the operand load: same bits
    return out, aux, dev, (W1b, W2b)


def per_token_errors(got, ref):
    """max |got - ref| / max |ref| of every token's output row."""
    den = np.abs(ref).max(axis=1)
    return np.abs(got - ref).max(axis=1) / np.where(den > 0, den, 1.0)


def test_config3_every_token(dyn, util, oracle):
    from workloads.rng import bf16_to_f32
    m = moe.config3()
    out, aux, dev, (W1b, W2b) = full_layer(dyn, util, m)
    ref_logits = oracle.moe_logits(m.x, m.Wg, m.Wn, m.noise)                         # (i) every logit
    assert util.normwise(aux["logits"], ref_logits) < LOGIT_TOL
    r = check_routing(oracle, m, aux)                                                # (ii) whole layer
    assert (r.counts[m.empty] == 0).all() and r.counts.sum() == m.A
    ref = oracle.moe_experts(m.x, r.topk_idx, r.topk_w, bf16_to_f32(W1b), bf16_to_f32(W2b))   # (iii) every token
    errs = per_token_errors(out, ref)
    assert errs.max() < OUT_TOL, (int(errs.argmax()), float(errs.max()))
    print(f"config 3: per-token error max {errs.max():.2e} median {np.median(errs):.2e}")
    load = np.sort(r.counts)[::-1].astype(np.float64)
    ok = load >= 8
    slope = np.polyfit(np.log(np.arange(1, m.E + 1)[ok]), np.log(load[ok]), 1)[0]
    assert abs(slope + 1.1) < 0.15


def config4_token_sample(r, k, min_tokens=512):
    """Tokens of config 4 whose output rows together touch every tile shape of the grouped expert layers:
    every use of 48 experts with fewer than 16 rows (one live 16-row sub-tile), of four experts with 17..63
    rows (two or four sub-tiles, ragged), and of the largest expert the first, a middle and the last 64-row
    tile (every fourth row plus the tile's first and last row); filled up with seeded random tokens."""
    counts, offsets, perm = r.counts, r.offsets, r.perm
    g = np.random.default_rng(4)
    pos = []
    tail = np.flatnonzero((counts > 0) & (counts < 16))
    tail = g.choice(tail, 48, replace=False)
    mid = np.flatnonzero((counts >= 17) & (counts <= 63))
    mid = np.concatenate([g.choice(mid[counts[mid] <= 32], 2, replace=False), g.choice(mid[counts[mid] > 32], 2, replace=False)])
    for e in np.concatenate([tail, mid]):
        pos += list(range(offsets[e], offsets[e + 1]))
    head = int(counts.argmax())
    n_tiles = (counts[head] + 63) // 64
    for tile in (0, n_tiles // 2, n_tiles - 1):
        lo = offsets[head] + 64 * tile
        hi = min(lo + 64, offsets[head + 1])
        pos += sorted(set(range(lo, hi, 4)) | {lo, hi - 1})
    tokens = set(int(perm[p]) // k for p in pos)
    T = len(r.topk_idx)
    while len(tokens) < min_tokens:
        tokens.add(int(g.integers(T)))
    return np.array(sorted(tokens)), dict(tail=tail, mid=mid, head=head, n_tiles=int(n_tiles))


def test_config4_targeted_tokens_with_empty_experts(dyn, util, oracle):
    from concurrent.futures import ThreadPoolExecutor
    m = moe.config4()
    out, aux, dev, (W1b, W2b) = full_layer(dyn, util, m)
    del W1b, W2b
    r = check_routing(oracle, m, aux)                                                # (ii) whole layer, bit-exact
    assert (r.counts[m.empty] == 0).all() and r.counts.sum() == m.A
    assert (np.sort(aux["perm"]) == np.arange(m.A)).all()
    assert (r.counts == 0).sum() >= 51 and len(m.empty) == 51
    tokens, info = config4_token_sample(r, m.k)
    assert len(tokens) >= 512 and len(info["tail"]) == 48 and info["n_tiles"] > 100
    ref_logits = oracle.moe_logits(m.x[tokens], m.Wg, m.Wn, m.noise[tokens])         # (i) the sampled rows
    assert util.normwise(aux["logits"][tokens], ref_logits) < LOGIT_TOL
    experts = np.unique(r.topk_idx[tokens])
    with ThreadPoolExecutor(16) as ex:                                               # weights regenerated per expert
        packs = dict(zip(experts.tolist(), ex.map(lambda e: m.expert_weights(int(e)), experts)))

    def one(t):
        es = [int(e) for e in r.topk_idx[t]]
        return oracle.moe_token(m.x[t], r.topk_w[t], [packs[e][0] for e in es], [packs[e][1] for e in es])

    with ThreadPoolExecutor(16) as ex:                                               # (iii) token by token
        ref = np.stack(list(ex.map(one, tokens)))
    errs = per_token_errors(out[tokens], ref)
    assert errs.max() < OUT_TOL, (int(tokens[errs.argmax()]), float(errs.max()))
    print(f"config 4: {len(tokens)} tokens through {len(experts)} experts, per-token error max {errs.max():.2e}")


@pytest.mark.parametrize("T,d,h,E,k,noise", [(1, 8, 8, 1, 1, True), (3, 40, 24, 5, 5, True), (17, 72, 136, 70, 2, False), (37, 512, 1024, 256, 2, False),
                                             (64, 1000, 520, 64, 8, True), (128, 64, 96, 64, 8, True), (129, 64, 64, 64, 8, False), (100, 64, 72, 4097, 2, True),
                                             (300, 48, 104, 40, 2, True), (700, 264, 520, 33, 2, True), (900, 1100 // 8 * 8, 64, 9, 3, False),
                                             (1200, 64, 16, 256, 1, True), (1201, 72, 16, 256, 1, False), (300, 64, 1024, 200, 2, False),
                                             (300, 1024, 64, 200, 2, False), (173, 384, 192, 5, 5, True), (160, 768, 96, 4, 2, False)])
def test_few_uses(dyn, util, oracle, T, d, h, E, k, noise):
    """The kernels for a few tokens, at the edges of their tiles (16 tokens, experts, features; 32 summed channels; rows of an
    expert up to and over 16, 32 and 64; blocks of 1024, 512 and 256 summed channels) and of their range (1200 gate tiles, 1024
    uses, 4096 experts; one expert layer on small tiles and the other not)."""
    m = moe.small(seed=T + E, T=T, d=d, h=h, E=E, k=k, zipf_s=1.1 if E < 1000 else 0.3)
    W1, W2 = stack(m)
    out, aux = util.moe_run(dyn, m, W1, W2, noise=noise)
    ref_logits = oracle.moe_logits(m.x, m.Wg, m.Wn if noise else None, m.noise if noise else None)
    assert util.normwise(aux["logits"], ref_logits) < LOGIT_TOL
    r = oracle.moe_route(aux["logits"], k)
    for name in ("topk_idx", "counts", "offsets", "perm", "inv"):
        assert (getattr(r, name) == aux[name]).all(), name
    ref = oracle.moe_experts(m.x, r.topk_idx, r.topk_w, W1, W2)
    assert per_token_errors(out, ref).max() < OUT_TOL


@pytest.mark.parametrize("T,d,h,E,k", [(4096, 1024, 2048, 8, 2), (8192, 512, 2048, 8, 2)])
def test_layers_of_full_tiles_keep_the_kernel_with_the_large_tiles(dyn, T, d, h, E, k):
    """The second layer has 2.8 rounds of workgroups of the kernel with the small tiles, whose row tiles each stream the weights for themselves:
    1.22 and 1.25 times the pass with the large tiles, which MOE_SEPARATE_PERMUTE always takes (and a launch more)."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(T)
    rnd = lambda *shape: (torch.randn(shape, generator=g, device="cuda") * 0.05).to(torch.bfloat16)
    args = (rnd(T, d), rnd(E, d), None, None, rnd(E, h, d), rnd(E, d, h), k)
    ws, out = torch.empty(dyn.moe_workspace_bytes(T, d, h, E, k), dtype=torch.uint8, device="cuda"), torch.empty_like(args[0])

    def ms(flags):
        start, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        start.record()
        for _ in range(20):
            dyn.moe_forward(*args, out=out, workspace=ws, flags=flags)
        end.record()
        end.synchronize()
        return start.elapsed_time(end)

    times = [(ms(0), ms(dyn.MOE_SEPARATE_PERMUTE)) for _ in range(7)][1:]
    assert min(t[0] for t in times) < 1.1 * min(t[1] for t in times), times


@pytest.mark.parametrize("T,E,k", [(1025, 7, 1), (1024, 4096, 2), (513, 300, 2), (8192, 40, 8), (8200, 33, 8), (600, 4097, 2), (2560, 4096, 8), (2561, 4096, 8),
                                   (9000, 1, 1), (65536, 1, 1), (1500, 2, 1), (700, 1024, 2), (2049, 1025, 2), (1300, 2051, 3)])
def test_grouping_of_many_uses(dyn, util, oracle, T, E, k):
    """Blocks of 1024 uses with a remainder of one, the most experts and uses of that path, and what lies beyond; a single expert, whose
    counts take all the room they have."""
    m = moe.small(seed=T + k, T=T, d=16, h=16, E=E, k=k, zipf_s=0.8)
    W1, W2 = stack(m)
    _, aux = util.moe_run(dyn, m, W1, W2)
    check_routing(oracle, m, aux)


def test_naive_per_use_loop_equals_batched_layer(dyn, util):
    """Results / MoE: the naive version loops over the k*b uses; same kernels, so the same bits as long as
    no group fills a 64-row tile (full tiles are multiplied with the 32x32x16 MFMA shape, which sums in
    another order)."""
    m = moe.small(seed=12, T=40, d=64, h=96, E=9, k=3, empty_frac=0.2)
    W1, W2 = stack(m)
    dev = util.moe_inputs_dev(m, W1, W2)
    a = dyn.moe_forward(dev["x"], dev["Wg"], dev["Wn"], dev["noise"], dev["W1"], dev["W2"], m.k)
    b = dyn.moe_forward(dev["x"], dev["Wg"], dev["Wn"], dev["noise"], dev["W1"], dev["W2"], m.k, naive_stride=1)
    assert (util.to_host(a) == util.to_host(b)).all()
    m2 = moe.small(seed=13, T=400, d=96, h=288, E=6, k=2)              # groups with full tiles: tolerance
    W1, W2 = stack(m2)
    dev2 = util.moe_inputs_dev(m2, W1, W2)
    a2 = dyn.moe_forward(dev2["x"], dev2["Wg"], dev2["Wn"], dev2["noise"], dev2["W1"], dev2["W2"], m2.k)
    b2 = dyn.moe_forward(dev2["x"], dev2["Wg"], dev2["Wn"], dev2["noise"], dev2["W1"], dev2["W2"], m2.k, naive_stride=1)
    assert util.normwise(util.to_host(a2), util.to_host(b2)) < 1e-2
    with pytest.raises(dyn.DynbError):
        dyn.moe_forward(dev["x"], dev["Wg"], dev["Wn"], dev["noise"], dev["W1"], dev["W2"], m.k, naive_stride=-1)


@pytest.mark.parametrize("h", [262144, 262408])
def test_naive_loop_over_experts_of_many_features(dyn, util, h):
    """1024 and 1026 feature tiles: one run of tiles for every XCD and two, the second one shorter.  The workspace is NaN before, so a
    tile left out would show.  Hidden units are rounded alike; the second layer's fp32 sums over h in another order and a rounding to
    bfloat16 (2^-9 of a value) differ."""
    import ctypes as ct
    import torch
    from paper_1707_02402_amd import binding
    g = torch.Generator().manual_seed(h)
    rnd = lambda *shape: torch.randn(shape, generator=g).to(torch.bfloat16).cuda()
    T, d, E = 3, 8, 2
    x, Wg, W1, W2 = rnd(T, d), rnd(E, d), rnd(E, h, d), rnd(E, d, h)
    shape = binding._MoeShape(T, d, h, E, 1, binding.DYNB_BF16, 0)
    ws = torch.full((int(binding.lib.moe_workspace_bytes(ct.byref(shape))),), 255, dtype=torch.uint8, device="cuda")
    a = dyn.moe_forward(x, Wg, None, None, W1, W2, 1)
    b = dyn.moe_forward(x, Wg, None, None, W1, W2, 1, workspace=ws, naive_stride=1)
    assert util.normwise(util.to_host(b), util.to_host(a)) < 1e-2


def test_moe_error_paths(dyn, util):
    import torch
    m = moe.small(seed=1, T=16, d=32, h=32, E=4, k=2)
    W1, W2 = stack(m)
    dev = util.moe_inputs_dev(m, W1, W2)
    with pytest.raises(dyn.DynbError) as e:
        dyn.moe_forward(dev["x"], dev["Wg"], dev["Wn"], dev["noise"], dev["W1"], dev["W2"], 5)
    assert e.value.name == "DYNB_E_INVAL"
    with pytest.raises(dyn.DynbError) as e:
        dyn.moe_forward(dev["x"], dev["Wg"], dev["Wn"], dev["noise"], dev["W1"], dev["W2"], 2,
                        workspace=torch.empty(256, dtype=torch.uint8, device="cuda"))
    assert e.value.name == "DYNB_E_WORKSPACE"
    with pytest.raises(dyn.DynbError) as e:
        dyn.moe_forward(dev["x"], dev["Wg"], None, dev["noise"], dev["W1"], dev["W2"], 2)
    assert e.value.name == "DYNB_E_INVAL"


def test_zero_tokens_is_a_successful_no_op(dyn):
    import torch
    d, h, E, k = 32, 32, 4, 2
    z = lambda *shape, dt=torch.bfloat16: torch.zeros(shape, dtype=dt, device="cuda")
    out = dyn.moe_forward(z(0, d), z(E, d), z(E, d), z(0, E, dt=torch.float32), z(E, h, d), z(E, d, h), k)
    assert out.shape == (0, d)


def test_every_token_to_one_expert_with_a_one_row_tail_tile(dyn, util, oracle):
    """k = 1 and one dominant gate column: a single group of 64*9 + 1 rows, every other group empty."""
    m = moe.small(seed=40, T=577, d=64, h=96, E=6, k=1)
    Wg = np.zeros_like(m.Wg)
    Wg[:, 4] = 0.0
    noise = np.full_like(m.noise, -8.0)
    noise[:, 4] = 8.0                                   # softplus(0) = ln 2: logit +-5.5, expert 4 always wins
    from dataclasses import replace
    m = replace(m, Wg=Wg, Wn=np.zeros_like(m.Wn), noise=noise)
    W1, W2 = stack(m)
    out, aux = util.moe_run(dyn, m, W1, W2)
    assert (aux["topk_idx"] == 4).all() and aux["counts"].tolist() == [0, 0, 0, 0, 577, 0]
    assert (aux["perm"] == np.arange(577)).all() and np.allclose(aux["topk_w"], 1.0)
    ref = oracle.moe_experts(m.x, aux["topk_idx"], aux["topk_w"], W1, W2)
    assert util.normwise(out, ref) < OUT_TOL


def test_layers_in_flight_on_three_streams(dyn, util):
    """Independent calls on their own streams, workspaces and outputs do not disturb each other.  The device is
    drained after the buffers are allocated: a side stream must not meet memory the default stream still uses."""
    import torch
    m = moe.config3()
    W1, W2 = stack(m)
    dev = util.moe_inputs_dev(m, W1, W2)
    args = (dev["x"], dev["Wg"], dev["Wn"], dev["noise"], dev["W1"], dev["W2"], m.k)
    ref = dyn.moe_forward(*args)
    nb = dyn.moe_workspace_bytes(m.T, m.d, m.h, m.E, m.k)
    lanes = [dict(s=torch.cuda.Stream(), ws=torch.empty(nb, dtype=torch.uint8, device="cuda"), out=torch.empty_like(ref))
             for _ in range(3)]
    torch.cuda.synchronize()
    for i in range(9):
        ln = lanes[i % 3]
        dyn.moe_forward(*args, out=ln["out"], workspace=ln["ws"], stream=ln["s"])
    torch.cuda.synchronize()
    for ln in lanes:
        assert torch.equal(ln["out"], ref)


def test_random_small_shapes(dyn, util, oracle):
    """Seeded sweep over ragged shapes (d, h multiples of 32 only; E and T arbitrary; k up to min(E, 8))."""
    g = np.random.default_rng(2024)
    for case in range(10):
        T = int(g.integers(1, 400))
        d = int(g.choice([32, 64, 96, 160, 288]))
        h = int(g.choice([32, 96, 224, 320]))
        E = int(g.integers(2, 140))
        k = int(g.integers(1, min(E, 8) + 1))
        m = moe.small(seed=1000 + case, T=T, d=d, h=h, E=E, k=k, empty_frac=float(g.choice([0.0, 0.3])))
        W1, W2 = stack(m)
        out, aux = util.moe_run(dyn, m, W1, W2)
        shape = (case, T, d, h, E, k)
        assert util.normwise(aux["logits"], oracle.moe_logits(m.x, m.Wg, m.Wn, m.noise)) < LOGIT_TOL, shape
        r = check_routing(oracle, m, aux)
        ref = oracle.moe_experts(m.x, r.topk_idx, r.topk_w, W1, W2)
        assert util.normwise(out, ref) < OUT_TOL, shape


@pytest.mark.parametrize("T,E,k", [(1, 1, 1), (1, 64, 8), (128, 8, 8), (1024, 3, 1), (1023, 2047, 1), (512, 257, 2), (513, 257, 1), (511, 2047, 2), (341, 1025, 3), (127, 2048, 8), (128, 2048, 8),
                                   (5, 2049, 2), (129, 300, 8), (114, 9, 9), (1024, 1, 1)])
def test_selection_and_grouping_in_one_launch_and_around_its_limits(dyn, util, oracle, T, E, k):
    """Up to 512 tokens, 1024 uses, eight of a token and 2048 experts the selection's last workgroup groups the uses; one use, expert or token beyond, launches of their
    own do.  Three passes over one workspace whose contents are arbitrary before the first: the counter is the layer's own affair."""
    import torch
    m = moe.small(seed=T + 3 * E + k, T=T, d=16, h=8, E=E, k=k, empty_frac=0.0)
    W1, W2 = stack(m)
    dev = util.moe_inputs_dev(m, W1, W2)
    ws = torch.full((dyn.moe_workspace_bytes(T, 16, 8, E, k),), 0xA5, dtype=torch.uint8, device="cuda")
    first = None
    for _ in range(3):
        out, aux = dyn.moe_forward(dev["x"], dev["Wg"], dev["Wn"], dev["noise"], dev["W1"], dev["W2"], k, want_aux=True, workspace=ws)
        aux = {n: v.cpu().numpy() for n, v in vars(aux).items()}
        check_routing(oracle, m, aux)
        first = util.to_host(out) if first is None else first
        assert (util.to_host(out) == first).all()
