"""The form of a generated kernel by its expression: an array read at several
sites asks for the block orders' geometry, an expression that reads every
array at one site does without it (it precedes the first load of every wave),
and a sum of two directions takes two waves of a group, not two of four, or in
FP32 with three fields around it stays a loop."""

import pytest

import paper_1105_2279_amd as q

FLAT = ["f0", "(add f0 (scale s0 f1))", "(umul 0 (shift f0 + 0))", "(shift (uadj 3 f0) - 3)",
        "(umul 3 (shift (umul 2 (shift f0 + 2)) + 3))", "(sum 0x8 (umul m (shift f0 + m)))",
        "(add (shift (shift f0 + 1) - 2) (shift (shift f0 - 2) + 1))"]
GEOMETRY = ["(add f0 (shift f0 + 1))", "(umul 1 (shift (umul 1 f0) + 1))", "(add (umul 0 f0) (shift (uadj 0 f1) - 0))",
            "(sub (sum 0x3 (umul m (shift f0 + m))) (sum 0x3 (shift (uadj m f0) - m)))",
            "(umul 2 (sum 0x5 (shift f0 + m)))"]
SPLIT = [("(sum 0x9 (umul m (shift f0 + m)))", 2), ("(add f1 (sum 0x6 (shift (uadj m f0) - m)))", 2),
         ("(sum 0x7 (umul m (shift f0 + m)))", 4), ("(scale s0 (sum 0xF (umul m (shift f0 + m))))", 4)]

MANY = [("(add (sum 0x3 (umul m (shift f0 + m))) (sub (scale s0 f1) (add f0 (shift f1 + 3))))", "jitgeo"),
        ("(add (sum 0x3 (umul m f1)) (sub (scale s0 f1) (add f1 f1)))", "flatgeo")]


@pytest.mark.parametrize("prec,fmt", [(q.F64, q.LINK18), (q.F32, q.LINK12)], ids=["f64", "f32_12"])
def test_kernel_form(prec, fmt):
    forms = [(e, 0, "flatgeo") for e in FLAT] + [(e, 0, "jitgeo") for e in GEOMETRY] + \
            [(e, n, "jitgeo") for e, n in SPLIT]
    forms += [(e, 2, "jitgeo") if prec == q.F64 else (e, 0, f32) for e, f32 in MANY]
    for e, split, geo in forms:
        src = q.jit_generate(e, prec, fmt, 2, 1)
        assert f"#define SPLIT {split}\n" in src, e
        assert f"int L3, {geo} geo," in src, e
