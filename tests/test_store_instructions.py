"""The store instructions of the built kernels (libkvx.so's own gfx950 code,
disassembled): which carry the streaming bit (nt) and which leave their pieces
to the L2 to merge."""
import os
import re
import shutil
import subprocess

import pytest

import paper_2509_17542_amd as K

LLVM = "/opt/rocm/llvm/bin"
TOOLS = [os.path.join(LLVM, t) for t in ("llvm-objcopy", "clang-offload-bundler", "llvm-objdump")]
pytestmark = pytest.mark.skipif(not all(shutil.which(t) for t in TOOLS),
                                reason="needs ROCm's LLVM tools")
QUANTISE = (2, 3, 12, 13)                        # kvx_internal.h, Conv: writes 8-bit codes
COPY8 = 4                                        # Conv: the 8-bit unpack
ALIGNED, FLAT, FLAT_CACHED = 0, 1, 2             # kvx_internal.h, Form


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """(operation, conversion, source order, form) -> its instructions."""
    d = tmp_path_factory.mktemp("isa")
    copy, fat, code = str(d / "lib.so"), str(d / "fat"), str(d / "code.o")
    subprocess.run([TOOLS[0], f"--dump-section=.hip_fatbin={fat}", K.LIB_PATH, copy], check=True)
    subprocess.run([TOOLS[1], "--unbundle", "--type=o", f"--input={fat}", f"--output={code}",
                    "--targets=hipv4-amdgcn-amd-amdhsa--gfx950"], check=True)
    text = subprocess.run([TOOLS[2], "-d", code], check=True, capture_output=True, text=True).stdout
    out = {}
    for part in re.split(r"\n(?=[0-9a-f]+ <)", text):
        m = re.match(r"[0-9a-f]+ <\S*kvx_(pack|unpack|repack)_kernelILi(\d+)ELi(\d)ELi(\d)E", part)
        if m:
            out[(m[1],) + tuple(int(x) for x in m.groups()[1:])] = \
                re.findall(r"^\t(\S.*?)\s*(?://|$)", part, re.M)
    return out


def _stores(code, name):
    return [i for i in code if i.startswith(name + " ")]


def _quantisers(kernels, *forms):
    pick = {k: v for k, v in kernels.items()
            if k[0] != "unpack" and k[1] in QUANTISE and k[3] in forms}
    assert len(pick) == 2 * len(QUANTISE) * 3 * len(forms)
    return pick


def test_scales_are_left_to_the_l2(kernels):
    """A wave's 4-byte row scales are pieces of sectors: never streamed by the
    quantisers and the flat unpack."""
    pick = _quantisers(kernels, ALIGNED, FLAT, FLAT_CACHED)
    pick.update({k: v for k, v in kernels.items()
                 if k[:2] == ("unpack", COPY8) and k[3] in (FLAT, FLAT_CACHED)})
    assert {k[0] for k in pick} == {"pack", "unpack", "repack"}
    for k, code in pick.items():
        scales = _stores(code, "global_store_dword")
        assert scales, k
        assert not [s for s in scales if re.search(r"\bnt\b", s)], (k, scales)


def test_rows_of_the_flat_forms(kernels):
    """16-byte row stores: streamed in the one flat form, ordinary in the other."""
    for form, streamed in ((FLAT, True), (FLAT_CACHED, False)):
        for k, code in _quantisers(kernels, form).items():
            rows = _stores(code, "global_store_dwordx4")
            assert rows and all(bool(re.search(r"\bnt\b", s)) == streamed for s in rows), (k, rows)


def test_unpack_does_not_wait_between_its_stores(kernels):
    """The 8-bit unpack's scale store follows the row's: a wait for loads in
    front of it would be one for the row's store too."""
    pick = {k: v for k, v in kernels.items() if k[:2] == ("unpack", COPY8)}
    assert {k[3] for k in pick} == {ALIGNED, FLAT, FLAT_CACHED}
    for k, code in pick.items():
        at = [i for i, c in enumerate(code) if c.startswith("global_store_dword ")]
        assert at, k
        for i in at:
            block = []              # from the branch or memory access before it
            while i and not re.match(r"s_c?branch|s_endpgm|global_", code[i - 1]):
                i -= 1
                block.append(code[i])
            assert not [c for c in block if "vmcnt" in c], (k, block)
