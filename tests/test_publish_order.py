"""The order in which the publish kernel's stores reach the host, read from its
AMD assembly: a host thread that sees the flag must see every word.  A missing
wait shows only now and then on a GPU, so it is looked for here."""
import os
import re
import subprocess

from paper_2606_20426_amd import build


def order_faults(asm):
    """What lets the flag (the store after the barrier) pass a word."""
    body = re.search(r"^\S*k_publish\S*:(.*?)s_endpgm", asm, re.S | re.M).group(1)
    code = [l.split(";")[0].strip() for l in body.splitlines()]
    code = [l for l in code if l and not l.endswith(":") and not l.startswith(".")]
    bar = max(i for i, l in enumerate(code) if l.startswith("s_barrier"))
    out = []
    words = [i for i, l in enumerate(code) if l.startswith("global_store") and i < bar]
    flags = [i for i, l in enumerate(code) if l.startswith("global_store") and i > bar]
    assert words and len(flags) == 1
    waits = [i for i, l in enumerate(code) if l.startswith("s_waitcnt") and "vmcnt(0)" in l]
    if not any(words[-1] < w < bar for w in waits):
        out.append("a wave reaches the barrier with stores under way")
    backs = [i for i, l in enumerate(code) if l.startswith("buffer_wbl2") and bar < i < flags[0]]
    if any(not any(b < w < flags[0] for w in waits) for b in backs):
        out.append("the flag does not wait for the write-back of the cache")
    for i in words + flags:
        if not re.search(r"\bsc0 sc1\b", code[i]):
            out.append("a store ends in the cache: " + code[i])
    return out


def test_words_reach_the_host_before_the_flag(tmp_path):
    asm = tmp_path / "publish.s"
    subprocess.run([build.hipcc(), *build.FLAGS, "--cuda-device-only", "-S", "-o", str(asm),
                    os.path.join(build.CSRC, "publish.hip")], check=True, stderr=subprocess.DEVNULL)
    assert order_faults(asm.read_text()) == []


def test_a_missing_wait_is_found():
    ok = """k_publish:
  global_store_dwordx2 v[4:5], v[6:7], off sc0 sc1
  s_waitcnt vmcnt(0)
  s_barrier
  buffer_wbl2 sc0 sc1
  s_waitcnt vmcnt(0)
  global_store_dwordx2 v2, v[0:1], s[4:5] sc0 sc1
  s_endpgm
"""
    assert order_faults(ok) == []
    wait = "  s_waitcnt vmcnt(0)\n"
    first, second = ok.index(wait), ok.rindex(wait)
    assert order_faults(ok[:first] + ok[first + len(wait):])
    assert order_faults(ok[:second] + ok[second + len(wait):])
    assert order_faults(ok.replace("off sc0 sc1", "off"))
