// The pair-coded form's dispatch (csrc/coded_kernels.hip) throws for operations and
// word counts it has no kernel for, before anything reaches a device.
#include "kernels.hpp"

#include <cstdio>
#include <stdexcept>

using namespace amg355;

template <class T>
static bool throws(RowOp op, CodedKind kind, int words) {
    static const uint32_t word = 0;
    CsrT<T> a{};
    a.rows = 256;
    a.pc_word = &word;
    a.pc_kind = kind;
    a.pc_words = words;
    T* const none = nullptr;
    try {
        launch_coded_op(op, a, none, none, none, T(0), none, none, DotTarget{nullptr, nullptr}, nullptr);
    } catch (const std::logic_error&) {
        return true;
    }
    return false;
}

int main() {
    int bad = 0;
    for (int words : {0, 7, 9, 17}) {
        for (CodedKind kind : {kCodedSquare, kCodedInterp, kCodedRestrict})
            for (RowOp op : {kSpmv, kResid, kJacobi, kSpmvAdd, kSpmvScale}) {
                bad += !throws<double>(op, kind, words);
                bad += !throws<float>(op, kind, words);
            }
    }
    for (int words : {2, 3, 8}) {
        for (RowOp op : {kSpmvAdd, kSpmvScale}) bad += !throws<double>(op, kCodedSquare, words) + !throws<float>(op, kCodedSquare, words);
        for (RowOp op : {kResidNorm, kJacobiDot, kSpmvDot}) bad += !throws<float>(op, kCodedSquare, words);
        for (RowOp op : {kSpmv, kResid, kJacobi, kSpmvScale, kSpmvDot}) bad += !throws<double>(op, kCodedInterp, words);
        for (RowOp op : {kResid, kJacobi, kSpmvAdd, kSpmvDot}) bad += !throws<double>(op, kCodedRestrict, words);
    }
    std::printf("%s\n", bad ? "dispatch: something went through" : "dispatch: ok");
    return bad != 0;
}
