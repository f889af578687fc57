"""The launches of a prompt product as planned on the host (nvq_gemm_describe)."""
import random

import pytest
import torch

from paper_2604_21026_amd import nvq

# (the planner assumes the device's compute units: the products of this file are cut at 256)
CUT = [(2049, 4104, 800), (2049, 4133, 800), (227, 4196, 11040), (1300, 3079, 2080), (1281, 3079, 2048),
       (4096, 6144, 4096)]


def launches(M, N, K, **kw):
    ls = nvq.gemm_describe(M, N, K, **kw)
    assert ls[0]["first_row"] == ls[0]["first_token"] == 0
    if len(ls) == 1:
        assert (ls[0]["rows"], ls[0]["tokens"]) == (N, M)
    elif ls[1]["first_row"]:      # cut by rows, in whole row tiles
        assert ls[1]["first_row"] == ls[0]["rows"] and ls[0]["rows"] + ls[1]["rows"] == N
        assert ls[0]["tokens"] == ls[1]["tokens"] == M and ls[0]["rows"] % ls[0]["tile_rows"] == 0
    else:
        assert ls[1]["first_token"] == ls[0]["tokens"] and ls[0]["tokens"] + ls[1]["tokens"] == M
        assert ls[0]["rows"] == ls[1]["rows"] == N and ls[0]["tokens"] % ls[0]["tile_tokens"] == 0
    return ls


@pytest.mark.parametrize("y_at", [0, 2, 8, 16])
def test_results_leave_16_bytes_at_a_time_only_where_every_address_is_aligned(y_at):
    rng = random.Random(5)
    drawn = [(rng.randint(33, 4096), rng.randint(256, 8192), 32 * rng.randint(16, 448)) for _ in range(400)]
    seen = set()
    for M, N, K in CUT + drawn + [(M, N // 8 * 8, K) for M, N, K in drawn]:
        for l in launches(M, N, K, dtype=torch.bfloat16, y_at=y_at):
            corners = [y_at + 2 * (m * N + n) for m in (l["first_token"], l["first_token"] + 1)
                       for n in (l["first_row"], l["first_row"] + l["rows"])]
            whole = all(a % 16 == 0 for a in corners)
            assert l["store_bytes"] == (16 if whole else 2), (M, N, K, l)
            seen.add((len(launches(M, N, K)), whole))
        assert all(l["store_bytes"] == 4 for l in launches(M, N, K))
    assert seen == ({(1, False), (2, False)} if y_at % 16 else {(1, False), (1, True), (2, False), (2, True)})
