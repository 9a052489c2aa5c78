"""The kernels that a call reaches only at certain sizes, alignments or options, at the sizes where
each can go wrong: edges of tiles and blocks, remainders, the smallest and the largest of a range."""
import gc

import numpy as np
import pytest

from oracle import gsq as ref
from paper_2604_18556_amd import binding as B

from gpu_common import Pair, assert_state_close, layer_inputs, oracle_params, rel_err

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B.load()
    return torch.device("cuda:0")


def _levels(K):
    return tuple(np.arange(K) - (K - 1) / 2.0)


# ------------------------------------------------------------------ state copies
# blocks of 1024 coordinates and of 16384: below one, at one, past one, and a ragged end
@pytest.mark.parametrize("O,I,gs", [(1, 16, 16), (4, 256, 128), (5, 208, 16), (65, 256, 64)])
@pytest.mark.parametrize("K", [2, 3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("shift", [0, 1])
def test_state_copies(dev, K, O, I, gs, shift):
    """set_state then get_state through pointers aligned to 16 bytes (shift 0) and to 4 only; the
    order inside is pinned by the hardened codes, which are numpy's argmax of the same logits."""
    W, H = layer_inputs(O, I, seed=K)
    rcfg = ref.Config(O, I, _levels(K), gs, precision="bf16", seed=3)
    layer = Pair(rcfg, W, H, dev).layer
    rng = np.random.default_rng(O * I + K)
    want = {n: rng.standard_normal((1, O, I, K)).astype(np.float32) for n in ("logits", "m", "v")}
    size = O * I * K
    bufs = {n: torch.zeros(size + 4, device=dev)[shift:shift + size] for n in want}
    for n in want:
        bufs[n].copy_(torch.from_numpy(want[n].reshape(-1)))
    layer.set_state(5, **bufs)
    out = {n: torch.full((size + 8,), 7.0, device=dev) for n in want}
    assert layer.get_state(**{n: x[shift:shift + size] for n, x in out.items()}) == 5
    for n, x in out.items():
        got = x.cpu().numpy()
        np.testing.assert_array_equal(got[shift:shift + size], want[n].reshape(-1))
        assert np.all(got[:shift] == 7.0) and np.all(got[shift + size:] == 7.0), "written outside"
    codes = torch.empty(1, O, I, dtype=torch.uint8, device=dev)
    layer.harden(codes=codes)
    np.testing.assert_array_equal(codes.cpu().numpy(), want["logits"].argmax(-1))


# ------------------------------------------------------------------ contraction
# (batch, O, I): every way the work is cut.  Tiles are 256 x 256; a last round of at most a
# quarter (half) of the 256 CUs is cut into quarters (halves).
@pytest.mark.parametrize("B_,O,I", [
    (1, 1, 16), (1, 129, 272), (1, 384, 640),       # quarters; 4 slabs and the shortest K loops
    (1, 300, 8256), (5, 300, 528),                  # quarters, ragged, over a batch
    (1, 1900, 3904), (17, 500, 512),                # halves only
    (1, 2048, 4352), (1, 4080, 4096),               # whole tiles only, below and at a round
    (1, 1000, 16400), (1, 5300, 4112),              # a whole round, then quarters; then halves
    (8, 2048, 1024), (9, 1800, 1008), (12, 2048, 1008),   # blocks: whole; a quartered; halved
    (10, 4200, 1040),                               # blocks that the last row of tiles does not fill
])
def test_contraction_cuts(dev, B_, O, I):
    """G = -2 R H of the library's own R against a float64 product of the same bf16 operands, and
    the hard loss against sum(R (R H)) of the hard residual, over the cuts of the work.

    Sums of I fp32 products in any order: an error of about 2^-24 sqrt(I) of the result's norm."""
    gen = torch.Generator(device=dev).manual_seed(O + I)
    W = (torch.randn(B_, O, I, generator=gen, device=dev) * 0.02).to(torch.bfloat16)
    X = torch.randn(B_, 512, I, generator=gen, device=dev)
    H = torch.stack([x.t() @ x for x in X])
    c = torch.tensor([-1.5, -0.5, 0.5, 1.5], device=dev, dtype=torch.float64)
    cfg = B.LayerConfig(O, I, tuple(c.tolist()), 16, batch=B_, seed=4)
    layer = B.Layer(cfg, W, H)
    layer.step(B.StepParams(tau=0.7))
    R = torch.empty(B_, O, I, device=dev, dtype=torch.bfloat16)
    G = torch.empty(B_, O, I, device=dev)
    layer.intermediates(R, G)
    codes = torch.empty(B_, O, I, dtype=torch.uint8, device=dev)
    scales = torch.empty(B_, O, I // 16, device=dev)
    hard = torch.zeros(B_, device=dev)
    layer.harden(codes=codes, scales=scales, hard_loss=hard)
    tol = 4 * 2.0 ** -24 * I ** 0.5
    for b in range(B_):
        Hb = ((H[b] + H[b].t()) * 0.5).to(torch.bfloat16).double()
        want = -2.0 * (R[b].double() @ Hb)
        err = (G[b].double() - want).norm() / want.norm()
        assert err <= tol, f"layer {b}: {err:.2e} > {tol:.2e}"
        worst = (G[b].double() - want).abs().max() / want.abs().max()
        assert worst <= 10 * tol, f"layer {b}: an element off by {worst:.2e}"
        q = c[codes[b].long()].float() * scales[b].repeat_interleave(16, 1)
        Rh = (W[b].float() - q).to(torch.bfloat16).double()
        loss = (Rh * (Rh @ Hb)).sum()
        assert abs(hard[b].double() - loss) <= max(tol, 2e-6) * loss, (b, hard[b].item(), loss.item())


# (batch, O, I) of the FP32 precision: 32 x 32 and 64 x 64 tiles, K slabs of 32, ragged ends
@pytest.mark.parametrize("B_,O,I", [(1, 1, 16), (1, 33, 48), (1, 256, 256), (3, 100, 208),
                                    (1, 1000, 1040), (2, 520, 1024), (1, 65, 16384)])
def test_contraction_fp32(dev, B_, O, I):
    """G = -2 R H of fp32 operands with fp64 sums, rounded once to fp32, and the hard loss."""
    gen = torch.Generator(device=dev).manual_seed(O + I)
    W = torch.randn(B_, O, I, generator=gen, device=dev) * 0.02
    X = torch.randn(B_, 64, I, generator=gen, device=dev)
    H = torch.stack([x.t() @ x for x in X])
    c = torch.tensor([-1.5, -0.5, 0.5, 1.5], device=dev)
    cfg = B.LayerConfig(O, I, tuple(c.tolist()), 16, batch=B_, seed=4, precision=B.PREC_FP32)
    layer = B.Layer(cfg, W, H)
    layer.step(B.StepParams(tau=0.7))
    R, G = torch.empty(B_, O, I, device=dev), torch.empty(B_, O, I, device=dev)
    layer.intermediates(R, G)
    codes = torch.empty(B_, O, I, dtype=torch.uint8, device=dev)
    scales = torch.empty(B_, O, I // 16, device=dev)
    hard = torch.zeros(B_, device=dev)
    layer.harden(codes=codes, scales=scales, hard_loss=hard)
    for b in range(B_):
        Hb = ((H[b] + H[b].t()) * 0.5).double()
        want = -2.0 * (R[b].double() @ Hb)
        # one rounding to fp32 of a sum whose fp64 error is far below it (|G| is not tiny next to
        # the terms: they are random)
        assert (G[b].double() - want).abs().max() <= 2.0 ** -23 * want.abs().max()
        Rh = (W[b] - scales[b].repeat_interleave(16, 1) * c[codes[b].long()]).double()
        loss = (Rh * (Rh @ Hb)).sum()
        assert abs(hard[b].double() - loss) <= 2e-6 * loss, (b, hard[b].item(), loss.item())


# ------------------------------------------------------------------ initialisation
# (relaxation, layout, levels, group): four coordinates per lane and 256 per wavefront, with ends
# inside a wavefront, and every group size
@pytest.mark.parametrize("relax,layout,K,gs", [
    ("grid", "group", 2, 16), ("grid", "group", 3, 32), ("grid", "group", 4, 64),
    ("grid", "group", 5, 128), ("grid", "group", 6, 256), ("grid", "group", 7, 16),
    ("grid", "group", 8, 128), ("grid", "superblock", 8, 16), ("shift", "group", 8, 64),
    ("shift", "group", 16, 16), ("ternary", "base3", 3, 32)])
@pytest.mark.parametrize("B_,O,units", [(1, 1, 1), (2, 5, 3), (1, 70, 5)])
@pytest.mark.parametrize("prec", ["bf16", "fp32"])
def test_initial_state(dev, relax, layout, K, gs, B_, O, units, prec):
    """Scales exactly, logits to their fp32 rounding (the noise's fp64 functions may differ by an
    ulp of fp64), base indices exactly; a zero group takes the scale 1 (0 in a super-block)."""
    I = units * (256 if layout == "superblock" else gs)
    W, H = layer_inputs(O, I, batch=B_, bf16=prec == "bf16", seed=K)
    W[-1, -1, -gs:] = 0.0
    rcfg = ref.Config(O, I, _levels(K), gs, batch=B_, precision=prec, seed=11, sigma_init=0.7,
                      relaxation=relax, layout=layout)
    got, st = Pair(rcfg, W, H, dev).get(), ref.init_layer(rcfg, W)
    np.testing.assert_array_equal(got.scales, st.scales)
    assert rel_err(got.logits, st.logits) <= 2.0 ** -23
    if relax == "shift":
        np.testing.assert_array_equal(got.base, st.base)
    assert not got.m.any() and not got.v.any() and not got.m_s.any() and not got.v_s.any()


@pytest.mark.parametrize("B_,I", [(1, 16), (2, 48), (1, 64), (1, 256), (3, 272), (1, 336)])
@pytest.mark.parametrize("prec", ["bf16", "fp32"])
def test_symmetrised_h(dev, prec, B_, I):
    """Rows of G = -2 R H for an H that is not symmetric: (H + H^T) / 2 is formed in fp32 and then
    rounded to the operand's type, over tiles of 64 with ragged ends."""
    gen = torch.Generator(device=dev).manual_seed(I)
    W = torch.randn(B_, 40, I, generator=gen, device=dev) * 0.02
    H = torch.randn(B_, I, I, generator=gen, device=dev)
    cfg = B.LayerConfig(40, I, _levels(4), 16, batch=B_, seed=4,
                        precision=B.PREC_FP32 if prec == "fp32" else B.PREC_BF16)
    dt = torch.float32 if prec == "fp32" else torch.bfloat16
    layer = B.Layer(cfg, W.to(dt), H)
    layer.step(B.StepParams(tau=0.7))
    R, G = torch.empty(B_, 40, I, device=dev, dtype=dt), torch.empty(B_, 40, I, device=dev)
    layer.intermediates(R, G)
    for b in range(B_):
        Hb = ((H[b] + H[b].t()) * 0.5).to(dt).double()
        want = -2.0 * (R[b].double() @ Hb)
        # fp32 sums of at most 336 products
        assert (G[b].double() - want).norm() <= 4 * 2.0 ** -24 * I ** 0.5 * want.norm()


# ------------------------------------------------------------------ fp64 backward
# one coordinate per lane, 256 columns per workgroup: groups inside a wavefront and across two and
# four, rows that end inside a wavefront, every number of Philox words per coordinate
@pytest.mark.parametrize("relax,K,gs,I", [
    ("grid", 2, 16, 16), ("grid", 2, 128, 384), ("grid", 3, 256, 512), ("grid", 4, 64, 320),
    ("grid", 5, 128, 128), ("grid", 5, 32, 96), ("grid", 6, 256, 256), ("grid", 7, 128, 640),
    ("grid", 7, 16, 272), ("grid", 8, 256, 768), ("shift", 8, 128, 384), ("shift", 16, 64, 64),
    ("ternary", 3, 128, 256), ("ternary", 3, 32, 288)])
@pytest.mark.parametrize("opt,samples", [(B.OPT_ADAM, 1), (B.OPT_LION, 1), (B.OPT_ADAM, 3)])
@pytest.mark.parametrize("loss", [True, False])
def test_fp64_steps(dev, relax, K, gs, I, opt, samples, loss):
    """Two steps, the second from the sample that the first drew, against the oracle: the same fp64
    arithmetic up to the order of sums, stored in fp32 (2^-24, and the same again in the second
    step's inputs).  A sign that flips within the rounding of a zero gradient is told apart."""
    W, H = layer_inputs(7, I, batch=2, bf16=False, seed=K)
    rcfg = ref.Config(7, I, _levels(K), gs, batch=2, precision="fp32", seed=5, relaxation=relax,
                      layout="base3" if relax == "ternary" else "group")
    pair = Pair(rcfg, W, H, dev)
    st = ref.init_layer(rcfg, W)
    rng = np.random.default_rng(I)
    st.m = (rng.standard_normal(st.m.shape) * 1e-3).astype(np.float32)
    st.v = (rng.uniform(0.5, 2, st.v.shape) * 1e-6).astype(np.float32)
    pair.put(st)
    for t in range(2):
        prm = B.StepParams(tau=0.6 - 0.1 * t, kappa=1.1, tau_next=0.5, kappa_next=1.1, optimizer=opt,
                           samples=samples, lr_scales=5e-5, weight_decay=0.01)
        got = pair.step(prm, want_loss=loss)
        st, want, inter = ref.step(rcfg, W, pair.Hs, st, oracle_params(prm), want=True)
        if loss:
            assert np.all(np.abs(got - want) <= 1e-6 * np.abs(want)), (t, got, want)
        assert_state_close(pair.get(), st, inter["G"], 1e-6, st.t, label=f"step {t}",
                           dlogits=inter["dlogits"])


# groups inside a wavefront, one wavefront, and across two and four
@pytest.mark.parametrize("gs", [16, 64, 128, 256])
@pytest.mark.parametrize("opt", [B.OPT_ADAM, B.OPT_LION])
@pytest.mark.parametrize("where,value", [("W", np.inf), ("W", np.nan), ("H", np.nan), ("H", -np.inf)])
def test_fp64_steps_with_values_that_are_not_finite(dev, gs, opt, where, value):
    """One weight or one diagonal element of H that is not finite makes a row or a column of G so.  A
    step without a loss sets the flag; each array of the state is finite just where the oracle's is
    and agrees there, so that the groups and wavefronts beside it are untouched.  Lion's step is a
    sign, which is 0 for NaN here and NaN in the oracle: its logits and scales stay finite."""
    W, H = layer_inputs(5, 512, batch=2, bf16=False, seed=gs)
    rcfg = ref.Config(5, 512, _levels(4), gs, batch=2, precision="fp32", seed=5)
    st = ref.init_layer(rcfg, W)
    if where == "W":
        W[1, 2, 300] = value
    else:
        H[1, 300, 300] = value
    pair = Pair(rcfg, W, H, dev)
    pair.put(st)
    prm = B.StepParams(tau=0.6, tau_next=0.6, lr_scales=5e-5, optimizer=opt)
    pair.step(prm, want_loss=False)
    with np.errstate(all="ignore"):
        st, _ = ref.step(rcfg, W, pair.Hs, st, oracle_params(prm))
    ls, ss = pair.shapes()
    got = {n: torch.empty(ls, device=dev) for n in ("logits", "m", "v")}
    got.update({n: torch.empty(ss, device=dev) for n in ("scales", "m_s", "v_s")})
    with pytest.raises(B.GsqError) as e:   # the state comes with the flag's report
        pair.layer.get_state(**got)
    assert e.value.status == B.GSQ_ENONFINITE
    for n in got:
        x, y = got[n].cpu().numpy(), getattr(st, n)
        fin = np.isfinite(y)
        assert fin[0].all() and fin[1].any() and not (n in ("m", "m_s") and fin[1].all()), n
        want = np.ones_like(fin) if opt == B.OPT_LION and n in ("logits", "scales") else fin
        np.testing.assert_array_equal(np.isfinite(x), want, err_msg=n)
        # m, v: 2^-24 of their size and the rounding of G; logits, scales: a step's size whatever the
        # gradient's, so the same of the step, next to which 1e-5 of the largest logit is wide
        assert np.abs(x[fin] - y[fin]).max() <= 1e-5 * np.abs(y[fin]).max(), n


# A launch holds fewer than 2^32 threads in a dimension: 2^24 - 1 of these kernels' workgroups.
def test_fp64_rows_beyond_one_grid_dimension(dev):
    """17 million rows of one workgroup each, past what one grid dimension holds: two steps (the
    second from the sample that the first drew) against the oracle on the rows at that edge and at
    the ends of the first and last layer."""
    B_, O, I, K = 5, 3_400_003, 16, 2
    edge = (1 << 24) - 1 - 4 * O   # in the last layer
    assert 0 < edge < O - 1
    rows = np.array([0, 1, edge - 1, edge, edge + 1, O - 1])
    print(f"[fp64 rows] {B_} x {O} x {I}", flush=True)
    gen = torch.Generator(device=dev).manual_seed(1)
    Wd = torch.randn(B_, O, I, generator=gen, device=dev) * 0.02
    X = torch.randn(B_, 64, I, generator=gen, device=dev)
    Hd = torch.stack([x.t() @ x for x in X])
    layer = B.Layer(B.LayerConfig(O, I, _levels(K), 16, batch=B_, precision=B.PREC_FP32, seed=5), Wd, Hd)
    # the oracle holds the sampled rows of the first and last layer, at their global noise indices
    rcfg = ref.Config(O, I, _levels(K), 16, batch=B_, precision="fp32", seed=5)
    W, Hs, sel = Wd.cpu().numpy(), ref.symmetrize(Hd.cpu().numpy())[[0, B_ - 1]], [0, B_ - 1]
    st = ref.init_layer(rcfg, W, rows=rows, batches=sel)
    big = torch.empty(B_, O, I, K, device=dev)
    for t in range(2):
        prm = B.StepParams(tau=0.6, tau_next=0.6, lr_scales=5e-5)
        loss = torch.full((B_,), -1.0, device=dev)
        layer.step(prm, loss_out=loss)
        st, _, inter = ref.step(rcfg, W, Hs, st, oracle_params(prm), rows=rows, batches=sel, want=True)
        got = {}
        for n in ("logits", "m", "v", "scales", "m_s", "v_s"):
            out = torch.empty(B_, O, 1, device=dev) if n in ("scales", "m_s", "v_s") else big
            tt = layer.get_state(**{n: out})
            got[n] = out[sel][:, rows].cpu().numpy()
        assert_state_close(ref.State(*got.values(), tt), st, inter["G"], 1e-6, t + 1,
                           label=f"step {t}", dlogits=inter["dlogits"])
        R, G = torch.empty(B_, O, I, device=dev), torch.empty(B_, O, I, device=dev)
        layer.intermediates(R, G)
        for b in range(B_):   # one partial per row, every one of them summed
            terms = R[b].double() * G[b].double() * -0.5
            assert abs(loss[b].double() - terms.sum()) <= 2.0 ** -23 * terms.abs().sum()
    layer.check()
    layer.destroy()
    B.release_cached()


# ------------------------------------------------------------------ memory kept between handles
@pytest.mark.parametrize("prec", ["bf16", "fp32"])
def test_layers_from_kept_memory(dev, prec):
    """A layer made of memory that other layers left behind gives the bits of the same layer made
    of fresh memory: shapes that fit the kept blocks exactly, with a margin, and not at all, with
    padding where the block's last user had data, on another stream, and with more samples."""
    def life(O, I, relax, stream=None, samples=1):
        W, H = layer_inputs(O, I, bf16=prec == "bf16", seed=O)
        rcfg = ref.Config(O, I, _levels(8), 16, precision=prec, seed=O, relaxation=relax)
        with torch.cuda.stream(stream or torch.cuda.current_stream()):
            pair = Pair(rcfg, W, H, dev)
            for t in range(2):
                loss = pair.step(B.StepParams(tau=0.9, tau_next=0.9, samples=samples))
            st, inter = pair.get(), pair.intermediates()
            codes = torch.empty(1, O, I, dtype=torch.uint8, device=dev)
            hard = torch.zeros(1, device=dev)
            pair.layer.harden(codes=codes, hard_loss=hard)
            out = [loss, st.logits, st.m, st.v, st.scales, *inter, codes.cpu().numpy(),
                   hard.cpu().numpy()]
            pair.layer.destroy()
        return out

    shapes = [(300, 272, "grid"), (256, 256, "grid"), (290, 272, "shift"), (40, 1040, "grid"),
              (512, 512, "grid"), (300, 272, "grid")]
    fresh = []
    for s in shapes:
        B.release_cached()
        fresh.append(life(*s))
    B.release_cached()
    other = torch.cuda.Stream()
    for n, k in enumerate([4, 0, 1, 2, 0, 3, 5, 0, 4, 2]):
        if n == 4:
            life(300, 272, "grid", samples=3)   # its larger G is left behind too
        for x, y in zip(life(*shapes[k], stream=other if n % 2 else None), fresh[k]):
            np.testing.assert_array_equal(x, y, err_msg=f"shape {shapes[k]}, use {n}")


def test_kept_memory_is_bounded_and_given_back(dev):
    """Ended handles keep at most a sixteenth of the device's memory; release_cached frees it."""
    gc.collect()   # what earlier tests left behind is not counted
    torch.cuda.empty_cache()
    B.release_cached()
    torch.cuda.synchronize()
    free0, total = torch.cuda.mem_get_info()
    H = torch.eye(256, device=dev).reshape(1, 256, 256)
    for O in (4096, 400_000, 4096):   # 8 levels: 27 MB per 1024 rows and array; 10 GB for the second
        W = torch.zeros(1, O, 256, device=dev, dtype=torch.bfloat16)
        layers = [B.Layer(B.LayerConfig(O, 256, _levels(8), 128), W, H) for _ in range(3)]
        for x in layers:
            x.destroy()
        del W, x, layers
        torch.cuda.empty_cache()
        kept = free0 - torch.cuda.mem_get_info()[0]
        assert kept <= total / 16 + (64 << 20), kept
    assert kept > 0
    B.release_cached()
    assert free0 - torch.cuda.mem_get_info()[0] <= 64 << 20


def test_kept_memory_goes_back_when_little_is_free(dev):
    """A handle that ends while less than an eighth of the device is free gives back its own memory and
    what earlier ones left: another allocator of the process holds the rest."""
    gc.collect()
    torch.cuda.empty_cache()
    B.release_cached()
    W = torch.zeros(1, 8192, 256, device=dev, dtype=torch.bfloat16)
    H = torch.eye(256, device=dev).reshape(1, 256, 256)
    free0, total = torch.cuda.mem_get_info()
    one, two = (B.Layer(B.LayerConfig(8192, 256, _levels(8), 128), W, H) for _ in range(2))
    one.destroy()
    free1 = torch.cuda.mem_get_info()[0]
    other = torch.empty(free1 - total // 10, device=dev, dtype=torch.uint8)
    print(f"[kept memory] {torch.cuda.mem_get_info()[0] >> 20} MiB free", flush=True)
    two.destroy()
    del other
    torch.cuda.empty_cache()
    assert free0 - torch.cuda.mem_get_info()[0] <= 64 << 20


# ------------------------------------------------------------------ loss reduction
# (batch, O, I): partials per layer below, at and past a chunk of 8192, several chunks, many layers
@pytest.mark.parametrize("B_,O,I", [(1, 1, 16), (1, 8191, 16), (1, 8192, 16), (1, 8193, 16),
                                    (3, 4100, 512), (70, 33, 272), (2, 30000, 256)])
def test_loss_reduction(dev, B_, O, I):
    """The step's loss against sum(-R G / 2) of the step's own R and G, several steps in a row (the
    hand-over between chunks is used again each time), and the same bits from gsq_step_static."""
    gen = torch.Generator(device=dev).manual_seed(O + I)
    W = (torch.randn(B_, O, I, generator=gen, device=dev) * 0.02).to(torch.bfloat16)
    X = torch.randn(B_, 64, I, generator=gen, device=dev)
    H = torch.stack([x.t() @ x for x in X])
    cfg = B.LayerConfig(O, I, _levels(4), 16, batch=B_, seed=4)
    one, two = B.Layer(cfg, W, H), B.Layer(cfg, W, H)
    R, G = torch.empty(B_, O, I, device=dev, dtype=torch.bfloat16), torch.empty(B_, O, I, device=dev)
    for t in range(4):
        prm = B.StepParams(tau=0.7, tau_next=0.7)
        la, lb = torch.full((B_,), -1.0, device=dev), torch.full((B_,), -2.0, device=dev)
        one.step(prm, loss_out=la)
        one.intermediates(R, G)
        two.step_static(prm, loss_out=lb)
        assert torch.equal(la, lb)
        want = (R.double() * G.double()).sum((1, 2)) * -0.5
        # fp32 sums of four columns' terms per lane (2^-24 each, of either sign) and one rounding
        size = (R.double() * G.double()).abs().sum((1, 2)) * 0.5
        assert torch.all((la.double() - want).abs() <= 2.0 ** -22 * size), (t, la, want)
