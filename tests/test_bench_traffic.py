"""The roofline's measured traffic belongs to the attention code that it was measured on."""
import json
import os
import shutil

import bench

CSRC = os.path.join(bench.ROOT, "paper_2604_22881_amd", "csrc")


def test_traffic_of_other_code_is_not_reported(tmp_path):
    path = tmp_path / "traffic.json"
    assert bench.measured_traffic(str(path)) is None
    path.write_text(json.dumps({"hbm_bytes_per_launch": 7}))
    assert bench.measured_traffic(str(path)) is None
    path.write_text(json.dumps({"hbm_bytes_per_launch": 7, "attention_sources": "0" * 64}))
    assert bench.measured_traffic(str(path)) is None
    path.write_text(json.dumps({"hbm_bytes_per_launch": 7, "attention_sources": bench.attention_sources_digest()}))
    assert bench.measured_traffic(str(path)) == 7


def test_digest_follows_the_code_and_not_its_comments(tmp_path):
    csrc = tmp_path / "csrc"
    shutil.copytree(CSRC, csrc)
    now = bench.attention_sources_digest()
    assert bench.attention_sources_digest(str(csrc)) == now
    kernel = csrc / "mts_attn_prefill.hip"
    text = kernel.read_text()
    kernel.write_text("// a word more\n" + text)
    (csrc / "mts_copy.hip").write_text("")
    assert bench.attention_sources_digest(str(csrc)) == now
    kernel.write_text(text.replace("constexpr int kTile = 32;", "constexpr int kTile = 16;"))
    assert bench.attention_sources_digest(str(csrc)) != now
