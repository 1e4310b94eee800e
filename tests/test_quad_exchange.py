"""The exchange of column sums between two waves of the embedding-gradient kernel at d = 128 (csrc/mfma_quad.hip, k_quad_dphi): its
order of barriers, reads and writes, replayed on the CPU from the kernel's text."""
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
COLUMNS = 16        # 128 / 8


def column_text():
    src = open(os.path.join(ROOT, "paper_2507_04239_amd", "csrc", "mfma_quad.hip")).read()
    kernel = src[src.index("void k_quad_dphi("):]
    return kernel[kernel.index("for (int tj = 0; tj < NB; ++tj)"):kernel.index("// the normaliser: rows of Gamma")]


def program():
    """(event, column) of one wave: barriers, the reads of both waves' sums of a column, the write of its own."""
    text = column_text()
    assert re.search(r"if \(i <= tj\) \{\s*lds_barrier\(\);", text)                         # one barrier per pair of tiles ...
    assert re.search(r"if \(i == 0\) \{[^}]*if \(RS == 2 && tj > 0\) land\(tj - 1\);", text)   # ... the sums behind the first
    write = text.index("hand[(w * 2 + tb) * 64 + lane] =")
    extra = re.search(r"if \((tj [=<>]+ \d+)\) lds_barrier\(\);\s*#pragma unroll[^;]*;[^;]*;[^;]*$", text[:write])
    out = []
    for tj in range(COLUMNS):
        for i in range(0, tj + 1, 2):
            out.append(("barrier", None))
            if i == 0 and tj > 0:
                out.append(("read", tj - 1))
        if extra and eval(extra.group(1), {"tj": tj}):
            out.append(("barrier", None))
        out.append(("write", tj))
    assert re.search(r"if constexpr \(RS == 2\) \{\s*lds_barrier\(\);\s*land\(NB - 1\);", text)
    return out + [("barrier", None), ("read", COLUMNS - 1)]


def test_a_barrier_lies_between_every_read_and_write_of_the_exchange():
    """The waves' accesses to one slot that are not ordered by the program of a wave itself are ordered by a barrier between: the
    write of a column before its reads, its reads before the next write."""
    epoch, reads, writes = 0, {}, {}
    for event, column in program():
        if event == "barrier":
            epoch += 1
        else:
            (reads if event == "read" else writes)[column] = epoch
    assert sorted(reads) == sorted(writes) == list(range(COLUMNS))
    for c in range(COLUMNS):
        assert writes[c] < reads[c], f"column {c}: read without a barrier behind its write"
        if c + 1 < COLUMNS:
            assert reads[c] < writes[c + 1], f"column {c}: its sums may be overwritten by column {c + 1}'s before the partner read them"
