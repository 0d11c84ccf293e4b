"""Kernels whose workgroups meet at barriers must leave a call as whole
workgroups.  Their waves read the control block's error word one by one, so
no workgroup of the same launch may write it: a late workgroup would
otherwise split, and the waves that stay would work from LDS that nobody
filled.  (Read from the source: a split depends on timing and cannot be shown
by running the kernels.)"""
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2609_09800_amd", "csrc")


def body(src, name):
    """Source text of the function `name`, up to the brace in column 0 that ends it."""
    at = re.search(r"\b%s\(" % name, src).start()
    return src[at:src.index("\n}\n", at)]


@pytest.mark.parametrize("file,exits,works", [
    ("hbf_blocking.hip", "k_regblock", "k_regblock"),
    ("hbf_kernels.hip", "k_cell_chan", "chan_units"),
])
def test_the_word_a_workgroup_leaves_on_is_not_written(file, exits, works):
    src = open(os.path.join(CSRC, file)).read()
    assert re.search(r"if \(.*ctl->err.*\) return;", body(src, exits))
    text = re.sub(r"//[^\n]*", "", body(src, exits) + body(src, works))
    assert not re.search(r"\batomic[A-Z]\w*\(&ctl->err\b|ctl->err\s*\|?=[^=]", text)


def test_the_cache_kernel_reads_its_status_once_per_workgroup():
    """Barriers that run out write the status word during the launch."""
    src = open(os.path.join(CSRC, "hbf_cache_chunk.hip")).read()
    text = re.sub(r"//[^\n]*", "", body(src, "k_chunk_run"))
    assert "st(status," in src
    reads = re.findall(r"[^;]*ld\(A\.status\)[^;]*;", text)
    assert len(reads) == 1 and "if (threadIdx.x == 0)" in reads[0]


def test_a_cache_call_that_runs_out_leaves_its_tags_behind():
    """Page words are told apart by the chunk's tag, which a reset does not
    clear: a call that ends at a barrier must not let the next one use its
    tags again, so every barrier of k_chunk_run passes the last tag on."""
    src = open(os.path.join(CSRC, "hbf_cache_chunk.hip")).read()
    text = re.sub(r"//[^\n]*", "", body(src, "k_chunk_run"))
    assert text.count("gr.sync()") == 1
    assert re.search(r"if \(gr\.sync\(\)\) return true;\s*if \(threadIdx\.x == 0\) atomicMax\(&cc\.ctl->epoch, epoch \+ 2\);", text)
