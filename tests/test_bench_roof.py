"""The roof that bench.py divides a stage by: the one that takes longer."""
import dataclasses

import bench
from paper_2601_05418_amd import synth


def test_fp32_contractions_meet_the_memory_roof_first():
    g = synth.highfield_slice(0).geom
    # W, a bank of 42 x 64 x 1024 and Z, 8 bytes each: 13 us at 8 TB/s against 5.9 us of products
    want = 8.0 * (32 * 224 * 1344 + 42 * 64 * 1024 + 42 * 64 * 224)
    for stage in ("group_compress", "group_expand"):
        assert bench.stage_roof(g, stage, "fp32") == ("hbm", want, "byte")
    assert bench.stage_roof(g, "readout_fwd", "fp32") == bench.stage_work(g, "readout_fwd", "fp32")
    # eight times the rows kept: the products bind
    wide = dataclasses.replace(g, k=512)
    assert bench.stage_roof(wide, "group_expand", "fp32") == bench.stage_work(wide, "group_expand", "fp32")
