"""The scalar slots that a kernel stores through FoldIn::scal and reads through its
restrict pointer to the same array: the compiler may take a slot read by the
latter as not written, so none may be both."""
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "paper_2012_11744_amd", "csrc", "pp_kernels.hip")

# slots that the shared helpers read from the array they are given
READS = {"set_alpha": {"S_ALPHA", "S_BETA", "S_USED", "S_RZNEW"}, "next_alpha": {"S_RZNEW", "S_USED"},
         "next_beta": {"S_RZOLD", "S_RZ", "S_DS", "S_USED"}, "new_rz": {"S_USED"}}


def function(text, name):
    start = re.search(r"\b%s\([^;{]*\)\s*\{" % name, text)
    depth, i = 1, start.end()
    while depth:
        depth += {"{": 1, "}": -1}.get(text[i], 0)
        i += 1
    return text[start.end():i]


def test_helpers_read_what_is_listed():
    text = open(SRC).read()
    for name, slots in READS.items():
        assert set(re.findall(r"\bscal\[(S_\w+)\]", function(text, name))) == slots, name


def test_no_slot_is_stored_and_read_through_different_pointers():
    text = open(SRC).read()
    for name in ("k_pcg_update", "direction_beta"):
        body = re.sub(r"//.*", "", function(text, name))
        stored = set(re.findall(r"in\.scal\[(S_\w+)\]\s*=", body))
        if "in.scal[q] = v" in body:          # set_alpha's setter
            stored |= set(re.findall(r"set\((S_\w+)", function(text, "set_alpha")))
        assert stored
        # the branch without folded sums stores nothing
        folded = body.split("else {")[0] if name == "k_pcg_update" else body.split("double v[1];")[1]
        read = set(re.findall(r"(?<!\.)\bscal\[(S_\w+)\]", folded))
        for call, args in re.findall(r"\b(set_alpha|next_alpha|next_beta|new_rz)\((.*)", folded):
            if re.search(r"(?<![.\w])scal\b", args):
                read |= READS[call]
        assert not (stored & read), (name, stored & read)
