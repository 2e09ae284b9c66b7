"""Which tile the GEMM takes where 128x128 and 256x192 are close: the larger one in bf16 from K = 4096 on."""
import pytest

from paper_2505_14468_amd import binding as B


@pytest.mark.parametrize("T,K,N,dtype,want", [(1380, 5120, 13824, 1, "tile_256x192"), (1764, 4096, 11008, 1, "tile_256x192"),
                                              (3830, 5120, 5120, 1, "tile_256x192"), (3830, 4088, 5120, 1, "tile_128x128"),
                                              (3184, 2048, 6000, 1, "tile_128x128"), (3830, 5120, 5120, 0, "tile_128x128"),
                                              (1350, 4096, 11008, 1, "tile_128x128")])
def test_tile_of_close_shapes(T, K, N, dtype, want):
    assert B.lora_gemm_kernel_name(None, T, K, N, dtype) == want
