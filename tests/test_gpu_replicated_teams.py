"""pp_plan_replicated from the bands in teams, around the lengths where three or four teams share a compute unit (768 and 1024
sets of eight orderings), against the oracle (bit for bit)."""
import pytest

import test_gpu_replicated_band as bands
from test_gpu_replicated import G  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seed,L,D,N,M,times", [
    (760, 32, 6, 6144, 29, 400), (761, 32, 6, 6145, 29, 400), (762, 32, 6, 7428, 29, 90), (763, 32, 6, 8192, 29, 400),
    (764, 32, 6, 8193, 29, 400), (765, 24, 8, 8000, 40, 60), (766, 40, 5, 6200, 16, 90)])
def test_teams(ppo, G, seed, L, D, N, M, times):  # noqa: F811
    bands.test_long_lists(ppo, G, seed, L, D, N, M, times)
