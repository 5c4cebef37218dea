"""Bound of an attention output against the float64 oracle, for the tests of the
attention's launch shapes (standard normal queries, keys and values).

An output of n keys has a norm of about 1/sqrt(n) of a value's, so a bound on its
elements does not see a missing block of keys once n is large; a bound relative to
each (row, head)'s own norm does: one key of n left out moves it by about
1/sqrt(n), 1.5e-2 at 4200 keys, and a block of 32 by 9e-2.  What the arithmetic
gives: probabilities rounded to fp16 (relative error up to 2^-11, independent from
key to key: about 3e-4 of the norm), outputs of parts of the keys in fp16 where
ranges are merged (2^-11 of an element: about 3e-4 as well), and for bf16 outputs
one rounding of up to 2^-9 of an element, 2e-3.  Hence 1e-3 for fp32 outputs and
5e-3 for bf16."""
import numpy as np

REL = {"f32": 1e-3, "bf16": 5e-3}


def worst_rel(got, ref):
    """Largest relative error (2-norms over the channels) of any (row, head)."""
    if got.size == 0:
        return 0.0
    err = np.linalg.norm(got.astype(np.float64) - ref, axis=-1)
    return float(np.max(err / np.linalg.norm(ref, axis=-1)))
