"""Order between the waves of a block, read off the kernels' source (no GPU):
what a run cannot be relied on to show, since the waves of a block usually
reach a word within a few cycles of each other.  Each test states the order
that the kernel needs and looks for the statement that makes it."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2603_07341_amd", "csrc")


def source(name):
    with open(os.path.join(CSRC, name)) as fh:
        text = fh.read()
    return re.sub(r"//[^\n]*", "", text)


def body(text, name):
    """Body of the function `name` (its first definition in `text`)."""
    for m in re.finditer(r"\b%s\s*\(" % name, text):
        at, depth = m.end(), 1
        while depth:
            depth += {"(": 1, ")": -1}.get(text[at], 0)
            at += 1
        rest = text[at:]
        if not rest.lstrip().startswith("{"):
            continue
        start = at = at + rest.index("{") + 1
        depth = 1
        while depth:
            depth += {"{": 1, "}": -1}.get(text[at], 0)
            at += 1
        return text[start:at - 1]
    raise AssertionError("no definition of " + name)


def test_top_pass_reads_need_before_the_block_that_writes_it():
    # the lane that finds the digit writes st->need, the waves that have not
    # searched yet must not read it any more
    b = body(source("cap.hip"), "k_top_pass")
    tail = b[b.index("last_block("):]
    reads = [m for m in re.finditer(r"st->need\b", tail)
             if not re.match(r"\s*=[^=]", tail[m.end():])]
    assert not reads, "read of st->need beside the write of the deciding lane"
    head = b[:b.index("last_block(")]
    assert "st->need" in head[:head.index("__syncthreads")]


def test_last_block_orders_every_wave_before_the_ticket():
    # a barrier waits for no global store or add of the other waves: each
    # wave waits for its own before the one that takes the ticket goes on
    text = source("common.hpp")
    b = body(text, "last_block")
    assert "stores_performed()" in b[:b.index("__syncthreads")]
    assert "vmcnt(0)" in body(text, "stores_performed")
    assert "__ATOMIC_ACQ_REL" in b and "MEMORY_SCOPE_AGENT" in b


def test_small_record_is_addressed_before_the_count_moves_on():
    # every wave finds the record by ctl->nrec, lane 0 increments it
    b = body(source("small.hip"), "small_observe")
    reads = [m.start() for m in re.finditer(r"ctl->nrec\b", b)]
    inc = b.index("ctl->nrec += 1")
    before = max(r for r in reads if r < inc)
    assert "__syncthreads()" in b[before:inc], "no barrier before the increment"


COLLECTIVE = r"__syncthreads|\bblock_\w+\s*\(|\bsums_\w+\s*\(|\blist_rows|_part<"


def kernels(text):
    """(name, parameters, body) of every kernel of a source."""
    for m in re.finditer(r"__global__\s+void\s+(?:__launch_bounds__\([^)]*\)\s*)?"
                         r"(k_\w+)\s*\(", text):
        b = body(text[m.start(1):], m.group(1))
        yield m.group(1), text[m.end():text.index(b, m.end())], b


def test_blocks_that_latch_read_the_latch_once():
    # kernels that can set the latch (err not const) while other blocks of
    # theirs start, and that use sums, scans or lists of the whole block
    seen = []
    for name in sorted(f for f in os.listdir(CSRC) if f.endswith(".hip")):
        for k, params, b in kernels(source(name)):
            if not re.search(r"(?<!const )int\s*\*\s*err\b", params):
                continue
            if not re.search(COLLECTIVE, b):
                continue
            seen.append(k)
            assert not re.search(r"if\s*\(\s*\*err\s*\)", b), (name, k)
            assert re.search(r"latched\(err\)|latch\s*=\s*\*err", b), (name, k)
    assert {"k_warm_probe", "k_warm_turn", "k_warm_list", "k_expand_probe",
            "k_expand_commit", "k_obs_final"} <= set(seen)


def test_small_expand_gathers_its_latch_in_lds():
    # any lane can meet an error, and the block goes on or stops by it: a
    # global add of another wave need not have landed by the next barrier
    b = body(source("small.hip"), "k_small_expand")
    for m in re.finditer(r"atomicOr\(a\.err", b):
        assert b[:m.start()].rstrip().endswith("if (threadIdx.x == 0)"), b[m.start() - 60:m.end()]
    assert "latch_now" not in b


def test_no_clear_runs_on_another_stream():
    # device memory is cleared on the stream that uses it: the null stream
    # does not order with the non-blocking streams that callers bring
    assert not re.search(r"\bhipMemset\s*\(", source("runtime.cpp"))
