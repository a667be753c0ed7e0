"""The placement of a ligand's pairs on batches and lanes decides the order of
every sum, so it may not change where only its computation does."""
import hashlib

import numpy as np
import pytest

from paper_2410_10447_amd import dock, synth

# first 16 digits of the SHA-256 of the exported batches
DIGESTS = {
    (1, 0): "e3b0c44298fc1c14", (12, 2): "316ca27a0eb1a639", (16, 4): "100f801af7539259",
    (17, 3): "7f9999313c6d1650", (32, 8): "6053d92b0ced276c", (33, 8): "954e1d116d16b1f1",
    (48, 10): "6dd2397f6b7e6376", (64, 16): "3fd42eac83440de0", (65, 12): "0127e7a024a7331a",
    (112, 28): "73a3891f77c6bb96", (128, 32): "e85374a02bac4142",
}


@pytest.mark.parametrize("atoms,torsions", sorted(DIGESTS))
def test_pairs_keep_their_batches_and_lanes(atoms, torsions):
    lig = dock.Ligand(synth.ligand(atoms, torsions, 104), synth.force_field(), upload=False)
    batches = np.ascontiguousarray(lig.export()["batches"])
    assert hashlib.sha256(batches.tobytes()).hexdigest()[:16] == DIGESTS[atoms, torsions]
