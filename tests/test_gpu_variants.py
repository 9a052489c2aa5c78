"""The kernels that a call reaches only at certain sizes, alignments or options, at the sizes where
each can go wrong: edges of tiles and blocks, remainders, the smallest and the largest of a range."""
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
