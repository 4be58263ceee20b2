"""Search at the sizes where its tiles end, against the oracle."""
import pytest
import torch

from tests import parity
from tests.test_gpu_parity_small import _gen, _run_search, ac  # noqa: F401

pytestmark = pytest.mark.gpu

VALU_CASES = [
    # N, E, B, k, dtype, metric: groups of 256 rows, slices of 32 columns, 4, 8 or 16 queries
    (1, 1, 1, 1, torch.float32, "ip"),
    (255, 31, 4, 1, torch.float32, "l2"),       # rows of odd length, one row short of a group
    (257, 33, 5, 3, torch.float32, "ip"),       # one column past a slice, one row past a group
    (2049, 45, 8, 1, torch.float32, "l2"),      # nine groups
    (513, 64, 9, 2, torch.float32, "l2"),
    (300, 768, 16, 1, torch.float16, "ip"),     # wider than the matrix-core kernels
    (4000, 40, 17, 4, torch.float16, "ip"),     # one query past a block
    (1000, 8, 33, 1, torch.float16, "l2"),
    (700, 1000, 3, 1, torch.float16, "l2"),
]


@pytest.mark.parametrize("case", VALU_CASES, ids=lambda c: "N%d-E%d-B%d-k%d-%s-%s" % (
    *c[:4], str(c[4]).split(".")[-1], c[5]))
def test_vector_alu_search_matches_the_oracle(ac, oracle_mod, case):  # noqa: F811
    N, E, B, k, dt, metric = case
    g = _gen(60 + N + E)
    emb = torch.randn(N, E, generator=g)
    emb = (emb / emb.norm(dim=1, keepdim=True)).to(dt)
    q = emb[torch.randint(0, N, (B,), generator=g)].float() + 0.02 * torch.randn(B, E, generator=g)
    q[::3] = torch.randn(q[::3].shape, generator=g) / E ** 0.5
    q = q.to(dt)
    m = ac.AC_IP if metric == "ip" else ac.AC_L2
    idx, score, hit = _run_search(ac, emb, q, k, 0.8, m)
    parity.check_search(oracle_mod, q, emb, k, 0.8, m, None, idx, score, hit)
