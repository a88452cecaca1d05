"""The argument types that binding.py gives to ctypes are those of the header, and wrong ones are refused."""
import os
import re

import pytest

import paper_2411_10803_amd as md
from paper_2411_10803_amd import binding

HEADER = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "include", "mustdrop.h")


def letter(param):
    if "*" in param:
        return "p"
    kind = param.split()[0]
    return {"int": "i", "int32_t": "i", "md_dtype": "i", "md_filter_mode": "i", "int64_t": "l", "float": "f", "size_t": "z"}[kind]


def test_signatures_match_the_header():
    with open(HEADER) as f:
        text = re.sub(r"/\*.*?\*/", "", f.read(), flags=re.S)
    found = {name: "".join(letter(p.strip()) for p in args.split(","))
             for name, args in re.findall(r"\bint (mustdrop_\w+)\(([^)]*)\);", text) if "*" in args}
    for name, sig in binding._SIGNATURES.items():
        assert sig == found[name], name


def test_wrong_argument_types_raise_type_error():
    for bad in (None, "7", 1.5):
        with pytest.raises(TypeError):
            binding._call("mustdrop_decode_append", *[None] * 8, bad, 1, 1, 8, 0, 1, None)
    with pytest.raises(md.MustDropError):                 # and right ones reach the library's own checks
        binding._call("mustdrop_decode_append", *[None] * 8, 1, 1, 1, 8, 0, 1, None)


def test_errors_of_a_conversion_itself_come_through():
    class Broken:
        def __float__(self):
            raise ValueError("no number")
    for bad, error in ((10 ** 400, OverflowError), (Broken(), ValueError), ("1.0", TypeError)):
        with pytest.raises(error):
            binding._call("mustdrop_decode_evict", *[None] * 7, 1, 1, 1, 8, bad, 1.0, 1, *[None] * 3, 0, None)
