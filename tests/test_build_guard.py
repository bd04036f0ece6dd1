"""Host logic of the build: what refuses kernels that use scratch memory, and unsafe wide stores."""
import os
import re

import pytest

from paper_2309_14717_amd import build as b

REMARK = """x.hip:1:1: remark: Function Name: {name} [-Rpass-analysis=kernel-resource-usage]
x.hip:1:1: remark:     VGPRs: 100 [-Rpass-analysis=kernel-resource-usage]
x.hip:1:1: remark:     ScratchSize [bytes/lane]: {scratch} [-Rpass-analysis=kernel-resource-usage]
"""


def test_clean_kernels_pass():
    text = REMARK.format(name="_ZN6qalora14gemm_dq_kernelILi4EEEv", scratch=0)
    b._check_no_scratch("gemm_dq.hip", text)


def test_spilling_kernel_is_refused():
    text = REMARK.format(name="_ZN6qalora14gemm_dq_kernelILi4EEEv", scratch=48)
    with pytest.raises(RuntimeError, match="scratch"):
        b._check_no_scratch("gemm_dq.hip", text)


def test_only_listed_kernels_are_checked():
    # another kernel of the same file may spill (it is not hand-scheduled)
    text = REMARK.format(name="_ZN6qalora12merge_kernelILi8EEEv", scratch=16)
    b._check_no_scratch("adapter.hip", text)
    text = REMARK.format(name="_ZN6qalora12front_kernelENS_9FrontArgsE", scratch=16)
    with pytest.raises(RuntimeError):
        b._check_no_scratch("adapter.hip", text)


@pytest.mark.parametrize("line,ok", [
    ("\tbuffer_store_dwordx4 v[28:31], v185, s[48:51], s12 offen sc1", False),
    ("\tbuffer_store_dwordx3 v[28:30], v185, s[48:51], m0 offen offset:16", False),
    ("\tbuffer_store_dwordx4 v[0:3], off, s[4:7], s0", False),
    ("\tbuffer_store_dwordx4 v[28:31], v185, s[48:51], 0 offen sc1", True),
    ("\tbuffer_store_dwordx2 v[28:29], v185, s[48:51], s12 offen", True),   # 64 bits: read at once
    ("\tbuffer_load_dwordx4 v[28:31], v185, s[48:51], s12 offen", True),
    ("\tglobal_store_dwordx4 v[0:1], v[2:5], off", True),
])
def test_wide_stores_with_a_scalar_offset_are_refused(line, ok):
    if ok:
        b._check_wide_stores("x.hip", line)
    else:
        with pytest.raises(RuntimeError, match="scalar offset"):
            b._check_wide_stores("x.hip", line)


def test_the_built_kernels_have_none():
    """The build checks what it compiles; this looks at the objects that are there."""
    objs = [os.path.join(b.OBJ, os.path.splitext(s)[0] + ".o") for s in b.SOURCES]
    if not all(map(os.path.exists, objs)):
        pytest.skip("not built here")
    stores = 0
    for src, obj in zip(b.SOURCES, objs):
        text = b._device_code(obj)
        b._check_wide_stores(src, text)
        stores += len(re.findall(r"buffer_store_dwordx4\b", text))
    assert stores > 0   # (the hand-over of partial sums: the listing is read as it should be)


def test_counted_waits_cover_the_lds_loads():
    """midt_kernel waits for x in LDS by counting: all but the newest n memory operations.  That covers the
    LDS loads only if at least n others were requested after the last of them."""
    obj = os.path.join(b.OBJ, "midt.o")
    if not os.path.exists(obj):
        pytest.skip("not built here")
    waits = 0
    for kernel in re.split(r"\n(?=[0-9a-f]+ <)", b._device_code(obj)):
        if "midt_kernel" not in kernel.split("\n", 1)[0]:
            continue
        lines = [ln.split("//")[0].strip() for ln in kernel.splitlines()]
        since = None   # memory operations since the last LDS load
        for ln, nxt in zip(lines, lines[1:]):
            if re.match(r"(buffer|global)_(load|store|atomic)", ln):
                since = 0 if ln.endswith(" lds") else (None if since is None else since + 1)
            m = re.match(r"s_waitcnt vmcnt\((\d+)\) lgkmcnt\(0\)", ln)
            if m and int(m.group(1)) > 0 and nxt == "s_barrier":
                assert since is not None and since >= int(m.group(1)), (lines[0], ln)
                waits += 1
    assert waits >= 2 * 21   # prologue and loop of every instantiation
