// What became of a unit of the resident pass, where the workgroups that see to units which gave up belong to the same launch: a word
// per unit, written by the unit and waited for by one of those workgroups.  No HIP in here: the host tests run it too.
#ifndef ADASUM_OUTCOME_H
#define ADASUM_OUTCOME_H

#ifdef __HIPCC__
#define ADASUM_ANYWHERE __host__ __device__ __forceinline__
#else
#define ADASUM_ANYWHERE inline
#endif

namespace adasum {

// kOverdue is no unit's word: what a wait comes back with that has ended without one.  (In forms with a second launch the word is a
// bare kGaveUp, and kRedone after that.)
constexpr int kOverdue = 0, kGaveUp = 1, kRedone = 2, kDone = 4;
ADASUM_ANYWHERE constexpr int outcome_word(unsigned tag, int what) { return static_cast<int>((tag - 1u) << 3) | what; }
ADASUM_ANYWHERE constexpr bool of_call(int word, unsigned tag) { return (word & 7) != 0 && word >> 3 == static_cast<int>(tag - 1u); }

// What became of a unit: kDone or kGaveUp, or kOverdue when `more` says no before that is known.
template <typename Load, typename More>
ADASUM_ANYWHERE int await_outcome(Load&& load, unsigned tag, More&& more) {
    for (;;) {
        const int word = load();
        if (of_call(word, tag)) return word & 7;
        if (!more()) return kOverdue;
    }
}

// What `load` says, for every wave of a workgroup alike: none goes on, and writes to what it reads, before all have looked.  (A branch
// with barriers in it hangs on the answer: a wave that saw a later one would leave the others waiting there.)
template <typename Load, typename Barrier>
ADASUM_ANYWHERE bool same_answer(Load&& load, Barrier&& barrier) {
    const bool answer = load();
    barrier();
    return answer;
}

}  // namespace adasum

#undef ADASUM_ANYWHERE
#endif
