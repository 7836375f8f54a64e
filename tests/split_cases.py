"""Sizes that reach every exponent of the parts of a cut row, and both sides of
the lengths past which rows are not cut (256 compute units), shared by the host
rule's test and the GPU's."""

# exponent -> values of one stream's row, cut into 129 parts of 2^exponent by
# every member, words and normals alike; the last part has 333 values.
EXPONENTS = {e: (1 << (e + 7)) + 333 for e in range(12, 21)}

# (streams or pairs of streams, values, parts, exponent): the longest rows that
# are cut, and one value more.
LONGEST = [(1, (1 << 28) + 255, 256, 20), (1, (1 << 28) + 256, 0, 0),
           (16, (1 << 26) + 255, 64, 20), (16, (1 << 26) + 256, 0, 0),
           (64, (1 << 24) + 255, 16, 20), (64, (1 << 24) + 256, 0, 0)]
