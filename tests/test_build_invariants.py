"""Properties of the generated gfx950 code that the attention kernel's hand-written LDS
transfers rely on (CPU only: hipcc cross-compiles the device code to assembly).

The transfer statement writes M0 itself and the kernel assumes that nothing else does:
no register-indirect indexing (v_movrel / s_movrel set M0), no other M0 user in between.
"""
import os
import re
import subprocess

import pytest

from paper_2503_16257_amd import build as B

SRC = os.path.join(B.CSRC, "decode_attn_mfma.hip")


def _isa(src, out):
    flags = [f for f in B.FLAGS if f not in ("-fPIC", "-Wall", "-Wno-unused-function")]
    cmd = [B._hipcc(), *flags, "-w", "-S", "--cuda-device-only", src, "-o", str(out)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return out.read_text()


@pytest.fixture(scope="module")
def attention_isa(tmp_path_factory):
    return _isa(SRC, tmp_path_factory.mktemp("isa") / "decode_attn_mfma.s")


def test_m0_is_written_only_by_the_transfer_statements(attention_isa):
    transfers = len(re.findall(r"^\s*global_load_lds_dwordx4\b", attention_isa, re.M))
    m0_lines = [l for l in attention_isa.splitlines() if re.search(r"\bm0\b", l) and not l.lstrip().startswith(";")]
    assert transfers > 0
    # every mention of M0 is the s_mov of one transfer statement
    assert all(re.match(r"\s*s_mov_b32 m0, s\d+", l) for l in m0_lines), \
        [l for l in m0_lines if not re.match(r"\s*s_mov_b32 m0, s\d+", l)][:5]
    assert len(m0_lines) == transfers
    assert "movrel" not in attention_isa


def test_no_register_spills_in_the_headline_variants(attention_isa):
    """n_a = 16 (the long-video and serving shapes), all three protected-row modes."""
    found = 0
    for m in re.finditer(r"\.name:\s+(\S+).*?\.vgpr_spill_count:\s+(\d+)", attention_isa, re.S):
        name, spills = m.group(1), int(m.group(2))
        if re.search(r"attn_mfma_kernelILi2ELi[012]ELb1E", name):
            found += 1
            assert spills == 0, (name, spills)
    assert found == 3


def test_residual_tokens_read_lds_16_bytes_at_a_time(tmp_path):
    """q and the probabilities come in quads only where the compiler knows their alignment."""
    isa = _isa(os.path.join(B.CSRC, "decode_attn.hip"), tmp_path / "decode_attn.s")
    m = re.search(r"^\S*attn_tail_kernel\S*:.*?s_endpgm", isa, re.S | re.M)
    assert len(re.findall(r"^\s*ds_read_b128\b", m.group(0), re.M)) >= 64
    assert not re.search(r"^\s*ds_read2", m.group(0), re.M)
