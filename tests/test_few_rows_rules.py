"""Which products of few rows add themselves to the residual rows: the rule at measured points on either side, on the CPU."""
import pytest
from test_abi_cpu import lib  # noqa: F401

F32, BF16 = 0, 1


# us per layer, K in shares / added
@pytest.mark.parametrize("d, K, rows, adds", [
    (2112, 2112, 8, True),                # 45.8 / 45.2
    (2112, 2112, 32, True),               # 62.3 / 61.2
    (4096, 4096, 17, True),               # 118.7 / 117.7
    (4352, 4352, 16, True),               # 149.2 / 149.1
    (4352, 4352, 17, False),              # 142.5 / 147.2
    (5120, 5120, 16, True),               # 174.9 / 173.7
    (5120, 5120, 24, False),              # 174.7 / 178.4
    (6144, 6144, 16, False),              # 227.4 / 227.3
    (8192, 8192, 8, True),                # 332.6 / 330.5
    (8192, 8192, 24, False),              # 368.6 / 370.0
    (2112, 8448, 5, False),               # 44.3 / 45.7
    (2112, 8448, 32, False),              # 61.2 / 65.7
    (2560, 10240, 8, False),              # 57.7 / 59.4
    (2560, 6912, 16, False),              # 58.8 / 60.8
    (3072, 12288, 16, False),             # 77.5 / 78.9
    (3584, 14336, 8, True),               # 86.4 / 85.9
    (3584, 14336, 17, False),             # 96.6 / 98.6
    (3840, 15360, 8, True),               # 93.5 / 92.0
    (3840, 15360, 12, False),             # 102.1 / 103.0
    (4096, 14336, 8, True),               # 117.4 / 116.4
    (4096, 16384, 24, True),              # 120.1 / 118.2
    (4096, 11008, 33, False),             # 40 rows: the activations cost more than the partial products
    (4352, 17408, 4, False),              # 121.7 / 125.5
    (5120, 13824, 8, False),              # 160.5 / 161.7
    (5120, 20480, 24, False),             # 178.4 / 194.6
    (8192, 32768, 8, True),               # 330.5 / 326.9
    (8192, 32768, 16, False),             # 357.2 / 363.0
    (1600, 1600, 17, True),               # 46.7 / 44.8
    (1600, 1600, 16, False),
    (1600, 6400, 24, False),              # 12.6 / 13.1, the product alone
    (768, 2048, 24, True),                # 32.4 / 32.0
    (256, 256, 24, False),                # 6.2 / 6.3, the product alone
])
def test_products_add_themselves_only_where_it_is_ahead(lib, d, K, rows, adds):  # noqa: F811
    rule = lib["_ZN8sprinter14gemm_adds_rowsEiiii"]
    assert bool(rule(BF16, d, K, rows) & 0xFF) == adds
    assert not rule(F32, d, K, rows) & 0xFF
