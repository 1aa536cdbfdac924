"""Which packs of a row the softmax kernels load and work on: exactly those that hold an allowed key.  The condition is read from
csrc/softmax.hip and compared with the definition over all alignments, lengths and limits, without a GPU."""
import os
import re

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2110_05722_amd", "csrc", "softmax.hip")


def test_a_pack_is_needed_where_it_holds_an_allowed_key():
    text = open(SRC).read()
    cond = re.search(r"bool pack_needed\(int j0, int limit\) \{ return (.*?); \}", text).group(1)
    expr = cond.replace("&&", " and ").replace("||", " or ").replace("!", " not ")
    for rag in (False, True):
        for s in range(8) if rag else (0,):                 # elements of the row's first pack in front of the row
            for k_len in range(1, 33) if rag else range(8, 33, 8):
                for limit in range(0, k_len + 1):           # 0: a padded query, an empty sentence or a row that does not exist
                    for idx in range((s + k_len + 7) // 8):
                        j0 = 8 * idx - s
                        want = any(0 <= j0 + j < limit for j in range(8))
                        assert bool(eval(expr, {"j0": j0, "limit": limit, "RAG": rag})) == want, (rag, s, k_len, limit, idx)
    # no load and no arithmetic of the kernels asks the limit in another way
    kernels = text[text.index("void softmax_fwd_kernel"):text.index("// ---- the same rows through LDS")]
    assert kernels.count("pack_needed<RAG>(") == 3 and not re.search(r"if \(j0 < limit\[r\]\)", kernels) and "__ballot(j0 < lim)" not in kernels
