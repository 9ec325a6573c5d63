"""Configuration names: the shipped table names what runs, and tables written
by earlier versions still load."""
import paper_2305_03448_amd as desc

EARLIER = {"gemm_grouped": "tile64_rm_d2", "transpose_32": "t128_nt_b512",
           "gemm_f32": "m128n128k16_rm_d2_x16", "gemm_bf16x3": "m256n256k32_w8d1_fused",
           "gemm_fp8": "m256n256k128_w8d1_p", "seg_reduce_i32": "unit32k",
           "seg_scan_i32": "unit8k"}


def _names(op):
    return [desc.desc_config_name(op, c) for c in range(desc.desc_config_count(op))]


def test_grouped_table_names_the_mixed_tiles():
    assert _names("gemm_grouped") == ["tile128_or_64", "tile64", "mixed128_64"]
    with open(desc.TUNE_FILE) as f:
        rows = [line.split()[2] for line in f if line.startswith("gemm_grouped ")]
    assert rows == ["mixed128_64"] * 4


def test_earlier_tables_load(tmp_path):
    path = tmp_path / "table.txt"
    path.write_text("".join(f"{op} {c} {name}\n" for op, name in EARLIER.items() for c in range(4)))
    try:
        assert desc.lib().desc_config_load(str(path).encode()) == 0
        for op, name in EARLIER.items():
            for c in range(4):
                got = _names(op)[desc.lib().desc_config_get(desc.OPS[op], c)]
                assert got == ("mixed128_64" if name == "tile64_rm_d2" else name)
    finally:
        for op in EARLIER:
            for c in range(4):
                desc.desc_config_set(op, c, -1)
