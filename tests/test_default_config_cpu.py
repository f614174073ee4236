"""The configuration a build takes unasked is the first of the ranked candidates, and
a geometry without candidates is refused by both, over sensors of all sizes and
maps of all turns.  Host code only; needs no GPU."""
import ctypes as C
import random

import numpy as np

import paper_2606_07759_amd as S
import workloads as wl


def test_default_is_the_first_candidate():
    lib = S.load()
    rng = random.Random(1)
    seen = set()
    for _ in range(150):
        p = rng.randint(1, 24)
        n_sub = rng.randint(1, max(1, min(90, 480 // p)))
        n = n_sub * p
        theta = (rng.uniform(-3, 3), rng.uniform(-3, 3),
                 rng.uniform(-3.2, 3.2) if rng.random() < 0.5 else rng.uniform(-0.05, 0.05),
                 rng.uniform(0.7, 1.4))
        A, _ = S.affine_from_misreg(theta, n + 20, n + 20, n, n)
        pupil = wl.pupil_mask(n, 2.0 * n)
        wfs = S.Wfs.from_numpy(pupil, p, wl.valid_subapertures(pupil, p), device="cpu").struct()
        a = S._affine_struct(A)
        one, all_, count = (C.c_int * 10)(), (C.c_int * 2560)(), C.c_int(0)
        status = lib.synim_im_config(C.byref(wfs), C.byref(a), one)
        assert lib.synim_im_candidates(C.byref(wfs), C.byref(a), all_, 256, C.byref(count)) == 0
        if status == 0:
            assert count.value > 0 and np.array_equal(list(one), list(all_[:10])), (n_sub, p, theta)
        else:
            assert count.value == 0, (n_sub, p, theta)
        seen.add(status)
    assert 0 in seen
