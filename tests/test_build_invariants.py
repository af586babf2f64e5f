"""Properties of the generated gfx950 code that the attention kernel's hand-written LDS
transfers rely on (CPU only: hipcc cross-compiles the device code to assembly).

The transfer statement writes M0 itself and the kernel assumes that nothing else does:
no register-indirect indexing (v_movrel / s_movrel set M0), no other M0 user in between.
"""
import concurrent.futures as cf
import os
import re
import subprocess

import pytest

from paper_2503_16257_amd import build as B

SOURCES = [f for f in B.SOURCES if f.startswith("decode_attn_mfma")]   # every instantiation of the kernel


def _isa(src, out):
    flags = [f for f in B.FLAGS if f not in ("-fPIC", "-Wall", "-Wno-unused-function")]
    cmd = [B._hipcc(), *flags, "-w", "-S", "--cuda-device-only", src, "-o", str(out)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return out.read_text()


@pytest.fixture(scope="module")
def attention_isa(tmp_path_factory):
    d = tmp_path_factory.mktemp("isa")
    with cf.ThreadPoolExecutor(max_workers=4) as ex:
        return dict(zip(SOURCES, ex.map(lambda f: _isa(os.path.join(B.CSRC, f), d / (f + ".s")), SOURCES)))


@pytest.mark.parametrize("src", SOURCES)
def test_m0_is_written_only_by_the_transfer_statements(attention_isa, src):
    isa = attention_isa[src]
    transfers = len(re.findall(r"^\s*global_load_lds_dwordx4\b", isa, re.M))
    m0_lines = [l for l in isa.splitlines() if re.search(r"\bm0\b", l) and not l.lstrip().startswith(";")]
    assert transfers > 0
    # every mention of M0 is the s_mov of one transfer statement
    assert all(re.match(r"\s*s_mov_b32 m0, s\d+", l) for l in m0_lines), \
        [l for l in m0_lines if not re.match(r"\s*s_mov_b32 m0, s\d+", l)][:5]
    assert len(m0_lines) == transfers
    assert "movrel" not in isa


def _states_before_first_transfer(lines):
    """Fewest wait states between the beginning of an assembly statement and a transfer with a scalar base, over
    its paths; None if a path has none."""
    labels = {l.rstrip(":"): i for i, l in enumerate(lines) if l.endswith(":")}
    best, todo = None, [(0, 0)]
    while todo:
        i, n = todo.pop()
        while i < len(lines):
            l = lines[i]
            if re.match(r"global_load_lds_dwordx4 v\d+, s\[", l):
                best = n if best is None else min(best, n)
                break
            if m := re.match(r"s_c?branch\S* (\S+)", l):
                todo.append((labels[m.group(1)], n + 1))
                if l.startswith("s_branch"):
                    break
            m = re.match(r"s_nop (\d+)", l)
            n += int(m.group(1)) + 1 if m else 0 if l.startswith(".") or l.endswith(":") else 1
            i += 1
    return best


@pytest.mark.parametrize("src", SOURCES)
def test_a_transfer_stands_five_wait_states_behind_its_statements_beginning(attention_isa, src):
    """A vector instruction may have written the scalar base right in front of the statement: then a memory
    instruction has to stand five wait states behind it, and the compiler does not look into the statement."""
    found = []
    for m in re.finditer(r"^\s*;;#ASMSTART$(.*?)^\s*;;#ASMEND$", attention_isa[src], re.S | re.M):
        lines = [l.split(";")[0].strip() for l in m.group(1).splitlines()]
        n = _states_before_first_transfer([l for l in lines if l])
        if n is not None:
            found.append(n)
    assert len(found) > 100 and min(found) >= 5, (len(found), min(found, default=None))


def test_no_variant_spills_vector_registers(attention_isa):
    """Every anomalous-channel count (n_a / 8 is the first template argument), the three protected-row
    modes, both key codes, without and with workgroups for residual tokens."""
    found = set()
    for isa in attention_isa.values():
        for m in re.finditer(r"\.name:\s+(\S+).*?\.private_segment_fixed_size:\s+(\d+).*?\.vgpr_spill_count:\s+(\d+)", isa, re.S):
            v = re.search(r"attn_mfma_kernelILi(\d+)ELi(\d)ELb(\d)ELb(\d)E", m.group(1))
            assert (m.group(2), m.group(3)) == ("0", "0"), m.groups()
            found.add(tuple(int(x) for x in v.groups()))
    both = {0, 1, 2, 4, 8, 12}                     # a variant without the residual part as well
    assert found == {(n, s, f, t) for n in range(17) for s in range(3) for f in (0, 1)
                     for t in ((0, 1) if n in both else (1,))}


def test_only_the_variants_with_an_inverse_dft_load_its_operands(attention_isa):
    """(Eq. 5 on at least one channel: the others would fetch 4 KB a workgroup and wait for it, and read none of it.)"""
    seen = set()
    for isa in attention_isa.values():
        for m in re.finditer(r"^_ZN\S*attn_mfma_kernelILi(\d+)ELi(\d)ELb(\d)ELb(\d)E\S*:.*?^\.Lfunc_end", isa, re.S | re.M):
            assert ("kIdftTab" in m.group(0)) == (m.group(3) == "1" and m.group(1) != "16"), m.groups()
            seen.add(m.groups())
    assert len(seen) >= 17 * 3 * 2


def test_residual_tokens_read_lds_16_bytes_at_a_time(tmp_path):
    """The value rows come through transposing reads, two for a tile of channels, and the waves' sums in quads, which
    they do only where the compiler knows their alignment.  (q and the probabilities, which this test looked at
    while the residual part ran on the vector ALU, are operands in registers.)"""
    isa = _isa(os.path.join(B.CSRC, "decode_attn.hip"), tmp_path / "decode_attn.s")
    m = re.search(r"^\S*attn_tail_kernel\S*:.*?s_endpgm", isa, re.S | re.M)
    reads = re.findall(r"^\s*(ds_read\w*)\b", m.group(0), re.M)
    assert set(reads) == {"ds_read_b128", "ds_read_b64_tr_b16"}
    assert reads.count("ds_read_b64_tr_b16") >= 16 and reads.count("ds_read_b128") >= 6
