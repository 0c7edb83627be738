"""What the library takes: hidden sizes up to 256 in every compiled shape and
size class, and the workspace size callers allocate (nep_loss_grad_noalloc
compares it with its 64 MiB scratch) for models of ordinary capacities: the
sum of the arrays of both lists' pair forces and reverse indices, however the
library lays out what it keeps.  Host functions only, no GPU."""
import random

import pytest

from paper_2507_00528_amd import nep

EXACT = [(2, 5, 5, 9, 9, 4, 0, 0), (2, 7, 5, 11, 11, 4, 2, 1), (2, 3, 2, 4, 3, 4, 2, 1), (1, 4, 3, 6, 5, 2, 2, 0),
         (2, 5, 4, 8, 8, 8, 2, 1)]
BAR_WORDS = 9 * 16     # the persistent step's barrier
PADDED = [(T, 12, 8, 12, 12, l, 2, 1) for l in (4, 8) for T in (1, 2, 3, 4)] + [(3, 4, 3, 6, 5, 4, 2, 1)]


def _model(shape, hidden, cap_rad=64, cap_ang=32):
    return nep.Model(*shape, hidden, 6.0, 4.0, cap_rad, cap_ang)


@pytest.mark.parametrize("shape", EXACT + PADDED)
def test_every_hidden_size_runs(shape):
    assert [H for H in range(1, 257) if not nep.model_supported(_model(shape, H))] == []


def _bytes(shape, hidden, cap_rad, cap_ang, S, N):
    """Arrays of 4-byte words: per atom position (padded to 32 atoms and 32 a
    species), per atom, per structure, and of fixed size."""
    T, NR, NA, KR, KA, L3, L4, L5 = shape
    pad = shape not in EXACT
    if pad:
        T, NR, NA, KR, KA, L3, L4, L5 = 4 if T > 2 else T, 12, 8, 12, 12, 8 if L3 > 4 else 4, 2, 1
    H, low = hidden, min(L3, 4)
    D = NR + NA * L3 + (NA if L4 else 0) + (NA if L5 else 0)
    YR, YH = 24 if low == 4 else 10, (L3 + 1) ** 2 - 25 if L3 > 4 else 0
    PW, TKR = T * NA * KA + 2 * H + 1, T * KR
    Np = ((N + 31) // 32 * 32 + T * 32 + 16 + 31) // 32 * 32
    N1, S1 = max(N, 1), max(S, 1)
    P = T * T * (NR * KR + NA * KA) + T * (H * D + 2 * H + 1) if pad else 0
    sizes = [4 * Np * k for k in (1, D, NA * YR, D, H, D, TKR, TKR, D if YH else NR, H, H, NA * YH, NA * YH)]
    sizes += [N1 * k for k in (4, 4 * cap_rad, 4 * cap_ang, 4, 12 * cap_rad, 12 * cap_ang, 24, 12, 12, 4, 4, 16)]
    sizes += [4 * S1, 24 * S1, 4 * S1, 24 * S1, 24 * S1, 16 * S1]
    sizes += [64, 4 * ((N1 + 1023) // 1024) * T * 64, 4 * (Np // 8) * PW, 8 * T * 512 * PW, 4 * T * 512 * H * D,
              4 * T * 256 * NR * TKR, 4 * (N1 + 1), 4 * (N1 // 2048 + 1), 128 * (N1 // 1024 + 1), 4, 4 * BAR_WORDS,
              1280, 4 * P, 4 * P, 4 * D * N1 if pad else 0]
    return sum((b + 255) // 256 * 256 for b in sizes)


def test_workspace_size_of_ordinary_capacities():
    rng = random.Random(5)
    for _ in range(4000):
        shape, H = rng.choice(EXACT + PADDED), rng.choice([1, 8, 16, 30, 50, 100, 256])
        cap_rad = rng.choice([16, 32, 64, 200])
        cap_ang = min(cap_rad, rng.choice([8, 16, 32]))
        N = int(2 ** rng.uniform(0, 22))
        S = max(1, int(N / 2 ** rng.uniform(0, 12)))
        case = (shape, H, cap_rad, cap_ang, S, N)
        assert nep.workspace_bytes(_model(shape, H, cap_rad, cap_ang), S, N) == _bytes(*case), case
