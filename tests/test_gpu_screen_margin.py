"""The margin that the basis builder stores with every seed's projector, read from the built stack:
it must cover what the fp16 rounding of the stored projector can take off the screen's form."""
import numpy as np
import pytest

from test_gpu_stream import sq  # noqa: F401
from test_screen_margin_host import I, J, MARGIN_A, SCALE, constant

pytestmark = pytest.mark.gpu


def _projector_section(sq, K, P):
    """fp16 [seeds of all tiles, 48 pairs] of a stack's projector section."""
    b = sq.build_bases(K, P)
    buf = b.buffer.cpu().numpy()
    seeds = (1 << K) - 1
    tile, pairs = int(constant("kSeedTile")), int(constant("kPairsPadded"))
    ntiles = -(-seeds // tile)
    # the stack's last section, but for the fp32 pseudo-inverses of P >= 5
    end = len(buf) - (-(-seeds * P * 8 * 4 // 256) * 256 if P >= 5 else 0)
    frag = buf[end - ntiles * tile * pairs * 2:end].view(np.float16)
    frag = frag.reshape(ntiles, 3, 2, tile, 8)   # fragment t, half h, seed, element e: pair 16 t + 8 h + e
    return frag.transpose(0, 3, 1, 2, 4).reshape(ntiles * tile, pairs)


@pytest.mark.parametrize("K", [8, 11])
@pytest.mark.parametrize("P", [1, 2, 3, 4, 5])
def test_stored_margin_covers_the_stored_rounding(sq, oq, K, P):  # noqa: F811
    got = _projector_section(sq, K, P)
    S, at = (1 << K) - 1, int(constant("kPairs"))
    assert not got[S:].any() and not got[:, at + 1:].any()
    U = oq.basis_int_all(K, P).astype(np.float64) * 2.0 ** -(K - 1)
    u, sv, _ = np.linalg.svd(U, full_matrices=False)
    keep = sv > 2.0 ** -30 * sv[:, :1]
    if (K, P) in ((11, 4), (11, 5)):
        assert not keep.all()   # rank-deficient seeds among them
    Pi = (u * keep[:, None, :]) @ u.transpose(0, 2, 1)
    a = got[:S, :at].astype(np.float64)
    want = SCALE * Pi[:, I, J]
    # half a unit of fp16 (2^-11, 2^-25 below its normal range), and the fp64 builder's error
    assert np.all(np.abs(a - want) <= 2.0 ** -11 * np.abs(want) + 2.0 ** -24)
    E = np.zeros((S, 8, 8))
    E[:, I, J] = E[:, J, I] = a - want
    norm = np.abs(np.linalg.eigvalsh(E)).max(1)
    # the margin's product with the block's operand, which is rounded to fp16 as well
    # (2^-11): in units of the form, MARGIN_A x kMarginScale = SCALE^2
    margin = got[:S, at].astype(np.float64)
    assert MARGIN_A * constant("kMarginScale") == SCALE ** 2
    assert np.all(margin * (1 - 2.0 ** -11) * SCALE / MARGIN_A >= norm)
    # and is no larger than ||E^2||_F^(1/2) asks for
    frob = np.sqrt(np.sqrt(((E @ E) ** 2).sum((1, 2))))
    assert np.all(margin * SCALE / MARGIN_A <= frob * (1 + 2.0 ** -7) + 2.0 ** -20)
