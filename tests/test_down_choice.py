"""The down projection's two weight blocks per wavefront, packed weights: where one each would make more than a round of workgroups (256 CUs) and
two make a single one, counted in the tiles that each form really has, a half-filled last one included, from 16 tiles of 256 features on; and beyond
192 rows per expert unless the launch is a single round of one block each even with the experts' second blocks.  Host arithmetic only."""
import pytest

import paper_2605_23911_amd as moe


def _two(T, d, E):
    moe.lib()
    name = moe.ffn_kernel_name(moe.MoEConfig.of(T, d, 4096, E, 1), 1, True)
    assert name.startswith(("tile_kernel_mixed<1, false, true, true", "tile_kernel_mixed<2, false, true, true"))
    return name.startswith("tile_kernel_mixed<2")


# rows per expert are few enough in every case that the other rules (512 workgroups of two blocks, rows per expert) do not speak
@pytest.mark.parametrize("d,E,two", [(4096, 16, True), (4096, 8, False), (6144, 8, True),       # 256 tiles of 256; 256 of 128; 192 of 256
                                     (4224, 15, True), (4224, 16, False),                       # 17 tiles: 255 and 272
                                     (4736, 13, True), (4736, 14, False),                       # 19 tiles: 247 and 266
                                     (4032, 16, False), (2688, 23, False), (2688, 24, False),   # 16 tiles and more, but not of 4096 features; 24 at 2688 are 504 of 128 and 264 of 256
                                     (640, 85, False), (640, 102, False)])
def test_one_round_of_two_blocks(d, E, two):
    assert _two(40 * E, d, E) == two


@pytest.mark.parametrize("T,d,E,two", [(192 * 16, 1024, 16, False), (193 * 16, 1024, 16, False), (239 * 16, 1024, 16, False),   # 8 tiles x (16 + 14)
                                       (192 * 16, 1280, 16, False), (193 * 16, 1280, 16, True),                                # 10 tiles x (16 + 12)
                                       (200 * 8, 2048, 8, False), (200 * 8, 2560, 8, True)])                                   # 16 and 20 tiles x (8 + 6)
def test_many_rows_per_expert(T, d, E, two):
    assert _two(T, d, E) == two
