"""Shapes that the 16-bit attention kernel deals to its workgroups in different ways: (way, B, H, W, L, D, longest context).
tests/test_attn_plan.py checks that the launch plan takes each of them the way named, tests/test_gpu_attn_dealing.py the results.

  ranked   more workgroups than the chip holds at once, eight tiles per wave and more, at most 64 sequences: longest first
  places   several row groups: as many workgroups as the packed rows take, their places found by a running sum
  in turn  several row groups, hundreds of sequences of short contexts: one workgroup per head takes its groups in turn
  heads    the same number of workgroups for every head
"""
SHAPES = [("ranked", 24, 22, 5, 3, 64, 1100), ("ranked", 24, 22, 12, 5, 64, 1150), ("ranked", 64, 9, 6, 2, 64, 1090),
          ("places", 64, 3, 12, 5, 64, 90), ("places", 70, 3, 12, 5, 128, 120), ("places", 257, 2, 17, 6, 64, 70), ("places", 515, 2, 12, 5, 64, 70),
          ("in turn", 300, 8, 12, 5, 64, 128), ("in turn", 530, 4, 17, 6, 64, 160), ("in turn", 700, 3, 10, 5, 128, 90),
          ("heads", 65, 9, 6, 2, 64, 1090), ("heads", 70, 8, 8, 5, 64, 1000)]
