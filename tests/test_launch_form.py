"""The form a call's iterations take, by its chains' number and lengths: the one
that measured faster, also where one chain is much longer than the others."""
import numpy as np
import pytest

import synth
from paper_1712_05012_amd import kcm

# residues of the chains and the launches of the faster form, each measured in
# both (mixed precision; 2 % or more of an iteration apart)
MEASURED = [
    ([15], 2), ([100], 2), ([200], 2), ([204], 2), ([250], 9), ([1000], 9),
    ([200] * 8, 2), ([300] * 8, 9), ([640] * 32, 9),
    ([15] * 4000, 2), ([30] * 4000, 2), ([15] * 3999 + [30], 2),
    ([210] * 128, 2), ([400] * 128, 2), ([300] * 256, 2),
    # one long chain, or some, among short ones
    ([15] * 127 + [200], 2), ([15] * 127 + [250], 2), ([15] * 127 + [400], 9), ([15] * 127 + [640], 9),
    ([15] * 255 + [300], 2), ([15] * 255 + [400], 9), ([15] * 255 + [640], 9),
    ([640] + [15] * 127, 9), ([15] * 112 + [640] * 16, 9), ([15] * 64 + [640] * 64, 9), ([60] * 120 + [400] * 8, 9),
    ([100] * 200 + [640], 9), ([100] * 200 + [400] * 56, 2),
    # and many very short ones beside one that takes a workgroup of 768 threads
    ([15] * 511 + [200], 2), ([2] * 511 + [200], 2), ([2] * 3999 + [60], 9), ([2] * 3999 + [200], 9),
    # the ragged batch of the benchmark
    (synth.batch_lengths(256, synth.config_seed(3)), 2),
    # longer than a workgroup holds
    ([641] * 128, 9),
]


@pytest.mark.parametrize("case", range(len(MEASURED)))
def test_form_is_the_one_that_measured_faster(case):
    n_res, launches = MEASURED[case]
    assert kcm.kcm_iteration_launches(n_res) == launches


def test_form_does_not_depend_on_the_order_of_the_chains():
    n_res = np.array([15] * 200 + [640] * 40 + [100] * 30, np.int32)
    for seed in range(4):
        assert kcm.kcm_iteration_launches(np.random.default_rng(seed).permutation(n_res)) == kcm.kcm_iteration_launches(n_res)


def test_form_rejects_bad_sizes():
    for bad in ([], [0], [5, (1 << 19) + 1]):
        with pytest.raises(kcm.KcmError) as e:
            kcm.kcm_iteration_launches(bad)
        assert e.value.status == kcm.KCM_E_INVAL
