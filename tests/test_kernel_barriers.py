"""Every workgroup barrier of the HIP sources is reached by all threads of a workgroup together:
none stands in a branch or loop whose condition differs between threads, and no thread leaves a
function that has a barrier further down.  Read from the sources (CPU)."""
import glob
import os
import re

import pytest

import conftest

CSRC = os.path.join(conftest.ROOT, "paper_2002_08816_amd", "csrc")
# names that differ between the threads of a workgroup in these sources
OWN = re.compile(r"\b(tid|threadIdx|lane|first|main|active|inmesh|hyb|on|tx|ty|lx|ly|gi|wv|myT|myH|q|it)\b")


def findings(text):
    """(line, statement) of the barriers that some threads of a workgroup may not reach."""
    text = re.sub(r"//[^\n]*|/\*.*?\*/", lambda m: re.sub(r"[^\n]", " ", m.group()), text, flags=re.S)
    out, stack, closed = [], [], None   # closed: the block that ended just before
    head = 0                            # start of the statement or block head being read
    for m in re.finditer(r"[{};]", text):
        h = re.sub(r"\s+", " ", text[head:m.start()]).strip()
        branch = re.match(r"(else )?(if|for|while)\b(?! constexpr)", h)
        own = bool(branch and OWN.search(h))
        k = max((i for i, b in enumerate(stack) if b["scope"]), default=-1)
        scope, here = (stack[k] if k >= 0 else dict(left=False)), stack[k + 1:]
        if m.group() == "{":
            if re.match(r"else\b", h) and closed and closed["own"]:
                own = True              # the other side of such a branch
            fn = "[&]" in h or bool(re.search(r"\)( const)?$", h) and not branch
                                    and not re.match(r"(else )?(if|switch|for|while)\b", h))
            stack.append(dict(own=own, scope=fn, left=False))
            closed = None
        elif m.group() == "}":
            closed = stack.pop() if stack else None
        else:
            split = own or any(b["own"] for b in here)
            if "__syncthreads" in h and (split or scope["left"]):
                out.append((text.count("\n", 0, m.start()) + 1, h))
            if re.search(r"\breturn\b", h) and split:
                scope["left"] = True
            closed = None
        head = m.end()
    return out


def test_the_reader_finds_both_kinds():
    ok = "void f() { int a; if (a) { __syncthreads(); } __syncthreads(); if (tid == 0) g(); } "
    assert not findings(ok)
    assert findings("void f() { int a; if (tid < 64) { __syncthreads(); } }")
    assert findings("void f() { int a; if (tid < 64) { a = 1; } else { __syncthreads(); } }")
    assert findings("void f() { int a; if (first) { a = 1; return; } __syncthreads(); }")
    assert findings("void f() { int a; if (first) return; __syncthreads(); }")


@pytest.mark.parametrize("path", sorted(glob.glob(os.path.join(CSRC, "*.hip")) + glob.glob(os.path.join(CSRC, "*.h"))),
                         ids=os.path.basename)
def test_barriers_are_met_by_all_threads(path):
    with open(path) as f:
        assert findings(f.read()) == []
