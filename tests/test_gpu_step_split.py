"""The matrix-core step of the generate kernels (and beside it the device
engine's) by every step size that they take, against the oracle's modular
product: random states, and states made from their successors so that the
carries at the end of the step run as far as they can."""
import random

import pytest
import torch

import oracle as O
import paper_2106_02504_amd as rlx
from rlx_util import ints_to_words, words_to_ints

pytestmark = pytest.mark.gpu

SPLIT_STEPS = 17  # up to 65 536 lanes per record


def successors():
    """Residues at the ends of the words that the last sums touch: 0, 1 and 7
    to 11 of the split form's, and the top word, all zeros or all ones."""
    top = (1 << 576) - 1
    out = [0, 1, 2, O.M - 1, O.M - 2, 1 << 288, (1 << 288) - 1, O.M >> 1]
    for lo, words in ((0, 2), (0, 7), (2, 5), (7, 3), (9, 2), (7, 11), (9, 9), (11, 7), (17, 1)):
        mask = ((1 << 32 * words) - 1) << 32 * lo
        for fill in (0x0123456789ABCDEF, 0xFEDCBA9876543210):
            base = sum(fill << 64 * k for k in range(9)) & top
            for low in (0, 1, (1 << 16) - 1, 1 << 16):
                out += [base | mask, base & ~mask, (base & ~mask) | low, (base | mask) ^ low]
    return [v % O.M for v in out]


@pytest.mark.parametrize("general", (False, True))
@pytest.mark.parametrize("p", (24, 2048))
def test_every_step_size(p, general):
    rng = random.Random(p)
    ys = successors()
    for g in range(SPLIT_STEPS):
        a = pow(O.multiplier(p), 2 ** g, O.M)
        inv = pow(a, -1, O.M)
        xs = [y * inv % O.M for y in ys] + ys + [rng.randrange(O.M) for _ in range(300)]
        x = torch.from_numpy(ints_to_words(xs)).cuda()
        got = words_to_ints(rlx.test_step(x, p, g, rlx.STEP_MFMA, general=general).cpu().numpy())
        assert got == [a * v % O.M for v in xs], (p, g)
